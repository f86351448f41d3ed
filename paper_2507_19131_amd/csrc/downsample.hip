// The layers between the stages of a Swin backbone (patch embedding, patch merging) as one
// uniformly quantized linear layer each: gather + (LayerNorm) + quantize + int8 MFMA +
// dequantize + (LayerNorm), one kernel.  The paper keeps these layers outside MixA-Q (its cost
// model lists them as the part the method cannot save, appendix on equivalent activation bits);
// they are here so that the four stages of a backbone run as one chain on the GPU.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/mixaq.h"
#include "mixaq_dev.h"
#include "arena.h"

namespace mixaq { int fail(int code, const char* fmt, ...); }
using namespace mixaq;

namespace {

struct DsArgs {
    const float* x;
    float* y;
    int B, H, W, Cin, P, K, Kp, N, Ho, Wo, tokens;
    FastDiv by_map, by_row;           // by Ho Wo, by Wo
    const v4i* Wp;                    // [N/32][Kp/32][64 lanes] x 16 bytes, natural k order, zero beyond K
    const float* m;                   // a_in.scale * s_w[n]
    const float* bias;                // [N] (zeros when the layer has none)
    const int* negcorr;               // -zp * sum_k W[n,k]
    const float* gamma;               // kind 0: [N], kind 1: [K]
    const float* beta;
    QDev q;
    float eps;
    int8_t* tap_codes;                // [tokens][K] or NULL
    int32_t* tap_acc;                 // [tokens][N] or NULL
};

__device__ __forceinline__ double sum8(double v)      // over the 8 lanes of a token
{
    v += __shfl_xor(v, 4, 64);
    v += __shfl_xor(v, 2, 64);
    v += __shfl_xor(v, 1, 64);
    return v;
}

// the four input values k0..k0+3 of output token (b,i,j); zero outside the map and beyond K
// (PC, CC: patch size and input channels when known at compile time, so that the index divisions are by constants; 0 = from A)
template <int KIND, int PC = 0, int CC = 0>
__device__ __forceinline__ float4 ds_values(const DsArgs& A, int b, int i, int j, int k0)
{
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (k0 >= A.K) return v;
    const int P = PC ? PC : A.P, Cin = CC ? CC : A.Cin;
    if (KIND == 1) {                  // 2x2 neighbours in the order (0,0), (1,0), (0,1), (1,1) [row, column offset]
        const int q = k0 / A.Cin, ch = k0 - q * A.Cin;
        const int r = 2 * i + (q & 1), c = 2 * j + (q >> 1);
        if (r < A.H && c < A.W) v = *(const float4*)(A.x + (((size_t)b * A.H + r) * A.W + c) * A.Cin + ch);
    } else {                          // patch values in the order (row in patch, column in patch, channel)
        float e[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int k = k0 + t, pc = k / Cin, ch = k - pc * Cin, di = pc / P, dj = pc - di * P;
            const int r = i * P + di, c = j * P + dj;
            e[t] = (r < A.H && c < A.W) ? A.x[(((size_t)b * A.H + r) * A.W + c) * Cin + ch] : 0.f;
        }
        v = make_float4(e[0], e[1], e[2], e[3]);
    }
    return v;
}

constexpr int MERGE_CUS = 256;                  // 8 XCDs of 32
// fragments in flight per wave: a part of the slabs that every split keeps whole
constexpr int merge_ring(int KS) { return KS % 3 == 0 ? (KS >= 48 ? 12 : 6) : 8; }
constexpr int merge_max_split(int KS) { return KS / merge_ring(KS) >= 4 ? 4 : 2; }

// Patch merging of the usual widths (C_in = LPT NV: 96, 128, 192, 256, 384, 512), one workgroup per 32 output tokens and
// per group of output blocks.
// Phase 1: LPT lanes per token, a quarter of them per neighbour, NV float4 each; the workgroup grows with C_in so that
// a lane's share of the 32 tokens is 48 or 64 floats, which it requests all at once: the kernel waits once for memory,
// and 128 registers leave room for sixteen waves per CU.  LayerNorm statistics in binary64 over the lane group, quantize,
// codes to LDS as MFMA operand fragments (slabs and halves a little apart, so that the lanes of a wave spread over the banks).
// Phase 2: wave w takes the output blocks first + w, first + w + waves, ... of its group; the weight fragments stream
// through a ring of loads in flight that starts before the barrier.  On a small grid `split` waves share the slabs of one
// output block (whole numbers: any order gives the same sums) and add up through LDS.  The tokens are the rows of the
// product and the output channels its columns, so a store writes whole 128-byte lines and a lane needs one m and one bias.
// Bound: memory on large maps (4 x 256 x 256 x 128: 59.4 -> 39.1 us on one map over and over, 65.5 -> 48.4 on fresh ones; before,
// 64 floats per lane and the hoisted gamma and beta took 224 registers, two waves per SIMD, and the vector unit idled two
// thirds of the time), the chain load - statistics - codes - products of one workgroup per CU on small ones (50 x 84 x 384:
// 21.2 -> 13.1 us).
template <int LPT, int NV, int NT, bool TAPS>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void merge_kernel(DsArgs A, int by_xcd, int groups, int per, int split)
{
    constexpr int CIN = LPT * NV, K = 4 * CIN, KS = K / 32, LQ = LPT / 4, TP = NT / LPT, PASSES = 32 / TP, NW = NT / 64;
    constexpr int RING = merge_ring(KS), HALF = 34, SLAB = KS % 16 == 0 ? 69 : 68;        // strides in 16-byte units
    static_assert(KS % RING == 0 && (LPT & (LPT - 1)) == 0 && LPT <= 64 && PASSES * NV <= 16, "lane groups inside a wave, whole ring turns");
    __shared__ v4i frag[(KS + 1) * SLAB];                     // one slab more: the operand of the step after the last is read, not used
    int* fragw = (int*)frag;
    int tile, group = 0;
    if (by_xcd) {                                             // the groups of a tile on one XCD: its inputs come through one L2
        const int slot = blockIdx.x >> 3;                     // (33 tiles of C_in = 384 in 6 groups: 3 of 15 us)
        tile = slot / groups * 8 + (blockIdx.x & 7);
        group = slot % groups;
        if (tile * 32 >= A.tokens) return;
    } else {
        tile = groups == 1 ? blockIdx.x : blockIdx.x / groups;
        group = groups == 1 ? 0 : blockIdx.x % groups;
    }
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    {
        const int grp = tid / LPT, q = (tid % LPT) / LQ, ch0 = (tid % LQ) * 4;
        float4 v[PASSES][NV];
        bool valid[PASSES], inside[PASSES];
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int tok = tile * 32 + p * TP + grp;
            valid[p] = tok < A.tokens;
            const int b = A.by_map(tok), rem = tok - b * A.by_map.d, i = A.by_row(rem), j = rem - i * A.by_row.d;
            const int r = 2 * i + (q & 1), c = 2 * j + (q >> 1);
            inside[p] = valid[p] && r < A.H && c < A.W;
            const float* src = A.x + (inside[p] ? (((size_t)b * A.H + r) * A.W + c) * CIN : 0) + ch0;
#pragma unroll
            for (int k = 0; k < NV; ++k) v[p][k] = *(const float4*)(src + k * (LQ * 4));
        }
        const float* gamma = A.gamma + q * CIN + ch0;
        const float* beta = A.beta + q * CIN + ch0;
        float mean[PASSES], rstd[PASSES];
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            if (!__all(inside[p])) {                          // the edge of an odd map, the last tile
#pragma unroll
                for (int k = 0; k < NV; ++k) {
                    v[p][k].x = inside[p] ? v[p][k].x : 0.f; v[p][k].y = inside[p] ? v[p][k].y : 0.f;
                    v[p][k].z = inside[p] ? v[p][k].z : 0.f; v[p][k].w = inside[p] ? v[p][k].w : 0.f;
                }
            }
            double s = 0.0, sq = 0.0;
#pragma unroll
            for (int k = 0; k < NV; ++k) s += sum4(v[p][k].x, v[p][k].y, v[p][k].z, v[p][k].w);
            mean[p] = ln_mean(lanes_sum<LPT>(s), K);
#pragma unroll
            for (int k = 0; k < NV; ++k) sq += centred4<true>(v[p][k].x, v[p][k].y, v[p][k].z, v[p][k].w, mean[p]);
            rstd[p] = ln_rstd(lanes_sum<LPT>(sq), K, A.eps);
        }
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const float4 gm = *(const float4*)(gamma + k * (LQ * 4)), bt = *(const float4*)(beta + k * (LQ * 4));
            const int k0 = q * CIN + ch0 + k * (LQ * 4);
#pragma unroll
            for (int p = 0; p < PASSES; ++p) {
                const int jt = p * TP + grp;
                const int code = pack4(quant_code(fmaf((v[p][k].x - mean[p]) * rstd[p], gm.x, bt.x), A.q), quant_code(fmaf((v[p][k].y - mean[p]) * rstd[p], gm.y, bt.y), A.q),
                                       quant_code(fmaf((v[p][k].z - mean[p]) * rstd[p], gm.z, bt.z), A.q), quant_code(fmaf((v[p][k].w - mean[p]) * rstd[p], gm.w, bt.w), A.q));
                if (TAPS && A.tap_codes && valid[p] && group == 0) *(int*)(A.tap_codes + (size_t)(tile * 32 + jt) * K + k0) = code;
                fragw[(((k0 >> 5) * SLAB + ((k0 & 31) >> 4) * HALF + jt) << 2) + ((k0 & 15) >> 2)] = code;
            }
            if (k & 1) __builtin_amdgcn_sched_barrier(0);     // not all of gamma and beta in registers at once
        }
    }
    const int j = lane & 31, g = lane >> 5, part = wave % split, len = KS / split;
    const int first = group * per, units = (min(first + per, A.N / 32) - first) * split;
    int nb = first + (wave < units ? wave / split : 0);
    const v4i* wp = A.Wp + ((size_t)nb * KS + part * len) * 64 + lane;
    v4i ring[RING];
#pragma unroll
    for (int d = 0; d < RING; ++d) ring[d] = wp[d * 64];
    __syncthreads();
    const v4i* fs = frag + part * len * SLAB + g * HALF + j;
    auto store = [&](const v16i& acc, float m, float bias) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int tok = tile * 32 + mfma_row(r, g);
            if (tok < A.tokens) {
                const size_t at = (size_t)tok * A.N + nb * 32 + j;
                A.y[at] = fmaf((float)acc[r], m, bias);
                if (TAPS && A.tap_acc) A.tap_acc[at] = acc[r];
            }
        }
    };
    v16i acc;
    for (int u = wave; u < units; u += NW) {                  // one turn where split > 1
        const float m = A.m[nb * 32 + j], bias = A.bias[nb * 32 + j];
        const int nc = part == 0 ? A.negcorr[nb * 32 + j] : 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = nc;
        const v4i* wnext = u + NW < units ? wp + (size_t)NW * KS * 64 : wp;               // behind the last turn: loaded, not used
        v4i f = fs[0];
#pragma unroll 1
        for (int k0 = 0; k0 < len; k0 += RING) {
            const v4i* wn = k0 + RING < len ? wp + (k0 + RING) * 64 : wnext;
#pragma unroll
            for (int d = 0; d < RING; ++d) {
                const v4i fn = fs[(k0 + d + 1) * SLAB];
                acc = mfma32(f, ring[d], acc);
                ring[d] = wn[d * 64];
                f = fn;
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (split == 1) {
            store(acc, m, bias);
            nb += NW;
        }
        wp = wnext;
    }
    if (split > 1) {                                          // uniform over the grid
        int* sums = (int*)frag + (wave / split * (split - 1) + (part ? part - 1 : 0)) * 1024 + lane;
        __syncthreads();                                      // the operand fragments have been read
        if (wave < units && part)
#pragma unroll
            for (int r = 0; r < 16; ++r) sums[r * 64] = acc[r];
        __syncthreads();
        if (wave < units && part == 0) {
            for (int t = 0; t < split - 1; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] += sums[t * 1024 + r * 64];
            store(acc, A.m[nb * 32 + j], A.bias[nb * 32 + j]);
        }
    }
}

// a load of four floats that need not lie on a 16-byte boundary (rows of 3 W floats do not)
typedef float f4_any __attribute__((ext_vector_type(4), aligned(4)));

// Patch embedding of 4x4x3 patches into 32 NB channels (96 and 128: the widths of Swin's first stages).  One wave per 32
// output tokens, nothing shared but the constants of the channels: lane = (token, half), a half holds two of the four patch
// rows (24 inputs in six loads of 16 bytes; the weights are packed in that order: 16 + 8 codes of each half
// and zeros), so the codes are MFMA operands where they were computed, and the 32 NB outputs of a token end in two lanes,
// whose LayerNorm sums need one exchange each.
// Bound: memory, once the map is large (4 x 1024 x 1024 into 128: with a tile's codes and outputs through LDS and three
// barriers 45.7 us on one image over and over and 63.1 on fresh ones, now 33.3 and 43.9, which is 4.2 TB/s); at 800 x 1344 into
// 96 (15.1 -> 11.0 us, fresh 18.8 -> 13.2) one chain of waits per wave, two waves per SIMD.  The 128 registers of four waves per
// SIMD need the two barriers against hoisting below.
template <int NB, bool TAPS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void embed_kernel(DsArgs A)
{
    constexpr int N = NB * 32;
    __shared__ float4 par[5][N / 4];                          // m, bias, gamma, beta, -zp * sum of the weights
    const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, g = lane >> 5;
    const int tok = (blockIdx.x * 4 + (tid >> 6)) * 32 + j;
    const bool valid = tok < A.tokens;
    const int b = A.by_map(tok), rem = tok - b * A.by_map.d, pi = A.by_row(rem), pj = rem - pi * A.by_row.d;
    float v[24];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int r = pi * 4 + g * 2 + h, c = pj * 4;
        const bool inside = valid && r < A.H;
        const bool whole = inside && c + 4 <= A.W;
        const float* row = A.x + (inside ? (((size_t)b * A.H + r) * A.W + c) * 3 : 0);
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const f4_any w = *(const f4_any*)((whole ? row : A.m) + t * 4);          // A.m: any 12 floats
            v[h * 12 + t * 4 + 0] = w.x; v[h * 12 + t * 4 + 1] = w.y; v[h * 12 + t * 4 + 2] = w.z; v[h * 12 + t * 4 + 3] = w.w;
        }
        if (!__all(whole)) {                                  // a patch over the edge of the map: pixel by pixel, zeros beyond
#pragma unroll
            for (int t = 0; t < 12; ++t) v[h * 12 + t] = inside && c + t / 3 < A.W ? row[t] : 0.f;
        }
    }
    v4i wf[NB][2];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) wf[nb][ks] = A.Wp[(nb * 2 + ks) * 64 + lane];
    for (int e = tid; e < 5 * (N / 4); e += 256) {
        const int which = e / (N / 4), at = e - which * (N / 4);
        const float* src = which == 0 ? A.m : which == 1 ? A.bias : which == 2 ? A.gamma : which == 3 ? A.beta : (const float*)A.negcorr;
        par[which][at] = ((const float4*)src)[at];
    }
    v4i code[2] = {};
#pragma unroll
    for (int t = 0; t < 6; ++t) {
        const int c = pack4(quant_code(v[t * 4 + 0], A.q), quant_code(v[t * 4 + 1], A.q), quant_code(v[t * 4 + 2], A.q), quant_code(v[t * 4 + 3], A.q));
        code[t >> 2][t & 3] = c;
        if (TAPS && A.tap_codes && valid) *(int*)(A.tap_codes + (size_t)tok * 48 + g * 24 + t * 4) = c;
    }
    __syncthreads();
    float f[NB * 16];
    double s = 0.0;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        __builtin_amdgcn_sched_barrier(0);                    // one block's constants and sums in registers at a time
        v16i acc;
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
            const int4 t4 = ((const int4*)par[4])[nb * 8 + qd * 2 + g];
            acc[qd * 4 + 0] = t4.x; acc[qd * 4 + 1] = t4.y; acc[qd * 4 + 2] = t4.z; acc[qd * 4 + 3] = t4.w;
        }
        acc = mfma32(wf[nb][0], code[0], acc);
        acc = mfma32(wf[nb][1], code[1], acc);
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
            const float4 m = par[0][nb * 8 + qd * 2 + g], bs = par[1][nb * 8 + qd * 2 + g];
            float* o = f + nb * 16 + qd * 4;
            o[0] = fmaf((float)acc[qd * 4 + 0], m.x, bs.x); o[1] = fmaf((float)acc[qd * 4 + 1], m.y, bs.y);
            o[2] = fmaf((float)acc[qd * 4 + 2], m.z, bs.z); o[3] = fmaf((float)acc[qd * 4 + 3], m.w, bs.w);
            s += sum4(o[0], o[1], o[2], o[3]);
            if (TAPS && A.tap_acc && valid)
                *(int4*)(A.tap_acc + (size_t)tok * N + nb * 32 + qd * 8 + g * 4) = make_int4(acc[qd * 4], acc[qd * 4 + 1], acc[qd * 4 + 2], acc[qd * 4 + 3]);
        }
    }
    const float mean = ln_mean(half_sum(s), N);
    double sq = 0.0;
#pragma unroll
    for (int k = 0; k < NB * 4; ++k) sq += centred4<NB != 3>(f[k * 4], f[k * 4 + 1], f[k * 4 + 2], f[k * 4 + 3], mean);
    const float rstd = ln_rstd(half_sum(sq), N, A.eps);
    if (!valid) return;
    float* out = A.y + (size_t)tok * N + g * 4;
#pragma unroll
    for (int k = 0; k < NB * 4; ++k) {
        if (k % 4 == 0) __builtin_amdgcn_sched_barrier(0);
        const float4 gm = par[2][k * 2 + g], bt = par[3][k * 2 + g];
        *(float4*)(out + k * 8) = make_float4(fmaf((f[k * 4 + 0] - mean) * rstd, gm.x, bt.x), fmaf((f[k * 4 + 1] - mean) * rstd, gm.y, bt.y),
                                              fmaf((f[k * 4 + 2] - mean) * rstd, gm.z, bt.z), fmaf((f[k * 4 + 3] - mean) * rstd, gm.w, bt.w));
    }
}

// The general form (patch embedding; patch merging of other widths).
// One workgroup (4 waves) per 32 output tokens.  Phase 1: eight lanes per token gather the K inputs
// (kind 1: LayerNorm over them, binary64 sums), quantize, and lay the codes out in LDS as MFMA
// operand fragments.  Phase 2: wave w computes the output blocks w, w+4, ...: W * codes^T, lane =
// token, 16 channels per block; dequantize; kind 1 stores, kind 0 goes through LDS for the
// LayerNorm over the N outputs of a token.
template <int KIND, int PC = 0, int CC = 0>
__global__ __launch_bounds__(256) void downsample_kernel(DsArgs A)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    v4i* frag = (v4i*)smem;                                   // [Kp/32][64]
    float* fo = (float*)(smem + (size_t)A.Kp * 32);           // kind 0: [32][N]
    int* fragw = (int*)smem;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    {
        const int jt = tid >> 3, sub = tid & 7;
        const int tok = blockIdx.x * 32 + jt;
        const bool valid = tok < A.tokens;
        const int b = tok / (A.Ho * A.Wo), rem = tok - b * (A.Ho * A.Wo), i = rem / A.Wo, j = rem - i * A.Wo;
        const int nch = A.Kp / 4, nreal = A.K / 4;
        float mean = 0.f, rstd = 1.f;
        if (KIND == 1) {
            double s = 0.0;
            if (valid)
                for (int c4 = sub; c4 < nreal; c4 += 8) {
                    const float4 v = ds_values<KIND, PC, CC>(A, b, i, j, c4 * 4);
                    s += ((double)v.x + (double)v.y) + ((double)v.z + (double)v.w);
                }
            s = sum8(s);
            mean = (float)(s / (double)A.K);
            double qv = 0.0;
            if (valid)
                for (int c4 = sub; c4 < nreal; c4 += 8) {
                    const float4 v = ds_values<KIND, PC, CC>(A, b, i, j, c4 * 4);
                    const double a0 = (double)v.x - (double)mean, a1 = (double)v.y - (double)mean;
                    const double a2 = (double)v.z - (double)mean, a3 = (double)v.w - (double)mean;
                    qv += (a0 * a0 + a1 * a1) + (a2 * a2 + a3 * a3);
                }
            qv = sum8(qv);
            const float var = (float)(qv / (double)A.K);
            rstd = 1.0f / sqrtf(var + A.eps);
        }
        for (int c4 = sub; c4 < nch; c4 += 8) {
            const int k0 = c4 * 4;
            int code = 0;
            if (valid && k0 < A.K) {
                float4 v = ds_values<KIND, PC, CC>(A, b, i, j, k0);
                if (KIND == 1) {
                    const float4 gm = *(const float4*)(A.gamma + k0), bt = *(const float4*)(A.beta + k0);
                    v.x = fmaf((v.x - mean) * rstd, gm.x, bt.x);
                    v.y = fmaf((v.y - mean) * rstd, gm.y, bt.y);
                    v.z = fmaf((v.z - mean) * rstd, gm.z, bt.z);
                    v.w = fmaf((v.w - mean) * rstd, gm.w, bt.w);
                }
                code = pack4(quant_code(v.x, A.q), quant_code(v.y, A.q), quant_code(v.z, A.q), quant_code(v.w, A.q));
                if (A.tap_codes) *(int*)(A.tap_codes + (size_t)tok * A.K + k0) = code;
            }
            // fragment (k slab, lane = half*32 + token): 16 bytes = the half's 16 consecutive k
            fragw[(((k0 >> 5) * 64 + ((k0 & 31) >> 4) * 32 + jt) << 2) + ((k0 & 15) >> 2)] = code;
        }
    }
    __syncthreads();
    const int j = lane & 31, g = lane >> 5, ksn = A.Kp / 32;
    const int tok = blockIdx.x * 32 + j;
    const bool valid = tok < A.tokens;
    for (int nb = wave; nb < A.N / 32; nb += 4) {
        v16i acc;
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
            const int4 t4 = *(const int4*)(A.negcorr + nb * 32 + qd * 8 + g * 4);
            acc[qd * 4 + 0] = t4.x; acc[qd * 4 + 1] = t4.y; acc[qd * 4 + 2] = t4.z; acc[qd * 4 + 3] = t4.w;
        }
        const v4i* wp = A.Wp + (size_t)nb * ksn * 64 + lane;
        for (int ks = 0; ks < ksn; ++ks) acc = mfma32(wp[ks * 64], frag[ks * 64 + lane], acc);
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
            const int n0 = nb * 32 + qd * 8 + g * 4;
            const float4 m = *(const float4*)(A.m + n0), bs = *(const float4*)(A.bias + n0);
            const float4 f = make_float4(fmaf((float)acc[qd * 4 + 0], m.x, bs.x), fmaf((float)acc[qd * 4 + 1], m.y, bs.y),
                                         fmaf((float)acc[qd * 4 + 2], m.z, bs.z), fmaf((float)acc[qd * 4 + 3], m.w, bs.w));
            if (valid && A.tap_acc) *(int4*)(A.tap_acc + (size_t)tok * A.N + n0) = make_int4(acc[qd * 4], acc[qd * 4 + 1], acc[qd * 4 + 2], acc[qd * 4 + 3]);
            if (KIND == 1) {
                if (valid) *(float4*)(A.y + (size_t)tok * A.N + n0) = f;
            } else {
                *(float4*)(fo + j * A.N + n0) = f;
            }
        }
    }
    if (KIND == 0) {                  // LayerNorm over the N outputs of a token, eight lanes per token
        __syncthreads();
        const int jt = tid >> 3, sub = tid & 7, tk = blockIdx.x * 32 + jt, nch = A.N / 4;
        const float* row = fo + jt * A.N;
        double s = 0.0;
        for (int c4 = sub; c4 < nch; c4 += 8) {
            const float4 v = *(const float4*)(row + c4 * 4);
            s += ((double)v.x + (double)v.y) + ((double)v.z + (double)v.w);
        }
        s = sum8(s);
        const float mean = (float)(s / (double)A.N);
        double qv = 0.0;
        for (int c4 = sub; c4 < nch; c4 += 8) {
            const float4 v = *(const float4*)(row + c4 * 4);
            const double a0 = (double)v.x - (double)mean, a1 = (double)v.y - (double)mean;
            const double a2 = (double)v.z - (double)mean, a3 = (double)v.w - (double)mean;
            qv += (a0 * a0 + a1 * a1) + (a2 * a2 + a3 * a3);
        }
        qv = sum8(qv);
        const float var = (float)(qv / (double)A.N);
        const float rstd = 1.0f / sqrtf(var + A.eps);
        if (tk < A.tokens)
            for (int c4 = sub; c4 < nch; c4 += 8) {
                const float4 v = *(const float4*)(row + c4 * 4);
                const float4 gm = *(const float4*)(A.gamma + c4 * 4), bt = *(const float4*)(A.beta + c4 * 4);
                *(float4*)(A.y + (size_t)tk * A.N + c4 * 4) =
                    make_float4(fmaf((v.x - mean) * rstd, gm.x, bt.x), fmaf((v.y - mean) * rstd, gm.y, bt.y),
                                fmaf((v.z - mean) * rstd, gm.z, bt.z), fmaf((v.w - mean) * rstd, gm.w, bt.w));
            }
    }
}

#define HIP_TRY(expr)                                                                                   \
    do {                                                                                                \
        hipError_t e_ = (expr);                                                                         \
        if (e_ != hipSuccess) return fail(MIXAQ_E_HIP, "%s failed: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

}  // namespace

struct mixaq_downsample {
    mixaq_downsample_desc d;
    int P = 0, K = 0, Kp = 0, Ho = 0, Wo = 0;
    FastDiv by_map, by_row;
    Arena mem;
    v4i* Wp = nullptr;
    float *m = nullptr, *bias = nullptr, *gamma = nullptr, *beta = nullptr;
    int* negcorr = nullptr;
    QDev q;
    ~mixaq_downsample() { mem.release(); }
};

namespace {

int ds_geometry(const mixaq_downsample_desc* d, int* P, int* K, int* Ho, int* Wo)
{
    if (!d) return fail(MIXAQ_E_NULL, "descriptor is NULL");
    if (d->kind != 0 && d->kind != 1) return fail(MIXAQ_E_SHAPE, "kind must be 0 (patch embedding) or 1 (patch merging)");
    if (d->B < 1 || d->H < 1 || d->W < 1 || d->C_in < 1) return fail(MIXAQ_E_SHAPE, "B, H, W, C_in must be positive");
    *P = d->kind == 0 ? d->patch : 2;
    if (*P < 1 || *P > 16) return fail(MIXAQ_E_SHAPE, "patch must be in 1..16");
    *K = *P * *P * d->C_in;
    if (*K % 4 != 0 || *K > 8192) return fail(MIXAQ_E_SHAPE, "inputs per token (%d) must be a multiple of 4, at most 8192", *K);
    if (d->kind == 1 && d->C_in % 4 != 0) return fail(MIXAQ_E_SHAPE, "patch merging needs C_in %% 4 == 0");
    if (d->N < 32 || d->N % 32 != 0 || d->N > 4096) return fail(MIXAQ_E_SHAPE, "N must be a multiple of 32 in 32..4096");
    if (d->act_bits < 2 || d->act_bits > 8 || d->weight_bits < 2 || d->weight_bits > 8)
        return fail(MIXAQ_E_BITS, "bit widths must be in 2..8");
    if (!(d->ln_eps > 0.0f)) return fail(MIXAQ_E_SHAPE, "ln_eps must be positive");
    *Ho = (d->H + *P - 1) / *P;
    *Wo = (d->W + *P - 1) / *P;
    if ((long long)d->B * *Ho * *Wo > (1LL << 30)) return fail(MIXAQ_E_SHAPE, "map too large for 32-bit token indexing");
    return MIXAQ_OK;
}

bool embed_in_registers(const mixaq_downsample_desc& d) { return d.kind == 0 && d.patch == 4 && d.C_in == 3 && (d.N == 96 || d.N == 128); }

size_t ds_lds_bytes(const mixaq_downsample* h) { return (size_t)h->Kp * 32 + (h->d.kind == 0 ? (size_t)32 * h->d.N * 4 : 0); }

int ds_forward(const mixaq_downsample* h, const float* x, float* y, void* stream, int8_t* tap_codes, int32_t* tap_acc)
{
    if (!h) return fail(MIXAQ_E_NULL, "handle is NULL");
    if (!x || !y) return fail(MIXAQ_E_NULL, "x or y is NULL");
    DsArgs A = {};
    A.x = x; A.y = y;
    A.B = h->d.B; A.H = h->d.H; A.W = h->d.W; A.Cin = h->d.C_in; A.P = h->P; A.K = h->K; A.Kp = h->Kp; A.N = h->d.N;
    A.Ho = h->Ho; A.Wo = h->Wo; A.tokens = h->d.B * h->Ho * h->Wo;
    A.by_map = h->by_map; A.by_row = h->by_row;
    A.Wp = h->Wp; A.m = h->m; A.bias = h->bias; A.negcorr = h->negcorr; A.gamma = h->gamma; A.beta = h->beta;
    A.q = h->q; A.eps = h->d.ln_eps; A.tap_codes = tap_codes; A.tap_acc = tap_acc;
    const dim3 grid((A.tokens + 31) / 32);
    const size_t lds = ds_lds_bytes(h);
    hipStream_t st = (hipStream_t)stream;
    const bool taps = tap_codes || tap_acc;
    // patch merging of the usual widths: the output blocks are split into groups while that leaves a CU of its own to each
    // workgroup, XCD by XCD (every group repeats phase 1, so a second workgroup on a CU costs more than the shorter phase 2
    // gives: 128 tiles of C_in = 96 in 2 groups 6.8 us, in 4 groups 9.2 us), and the slabs of a block over the waves that have
    // no block of their own
#define MERGE_CASE(L, V, NT)                                                                                          \
    if (h->d.kind == 1 && A.Cin == L * V) {                                                                           \
        const int NB = A.N / 32, tiles = (int)grid.x;                                                                 \
        const int room = tiles < 8 ? MERGE_CUS / tiles : MERGE_CUS / 8 / ((tiles + 7) / 8);                           \
        const int most = std::max(1, std::min(NB, room)), per = (NB + most - 1) / most, groups = (NB + per - 1) / per;  \
        int split = 1;                                                                                                \
        while (split < merge_max_split(L * V / 8) && per * split * 2 <= NT / 64) split *= 2;                          \
        const int by_xcd = tiles >= 8 && groups > 1;                                                                  \
        const dim3 grid2((by_xcd ? (tiles + 7) / 8 * 8 : tiles) * groups);                                            \
        if (taps) hipLaunchKernelGGL((merge_kernel<L, V, NT, true>), grid2, dim3(NT), 0, st, A, by_xcd, groups, per, split); \
        else hipLaunchKernelGGL((merge_kernel<L, V, NT, false>), grid2, dim3(NT), 0, st, A, by_xcd, groups, per, split);   \
        HIP_TRY(hipGetLastError());                                                                                   \
        return MIXAQ_OK;                                                                                              \
    }
    MERGE_CASE(32, 3, 256) MERGE_CASE(32, 4, 256) MERGE_CASE(64, 3, 512) MERGE_CASE(64, 4, 512) MERGE_CASE(64, 6, 1024) MERGE_CASE(64, 8, 1024)
#undef MERGE_CASE
    if (embed_in_registers(h->d)) {
        const dim3 grid4((A.tokens + 127) / 128);
        if (A.N == 96) {
            if (taps) hipLaunchKernelGGL((embed_kernel<3, true>), grid4, dim3(256), 0, st, A);
            else hipLaunchKernelGGL((embed_kernel<3, false>), grid4, dim3(256), 0, st, A);
        } else {
            if (taps) hipLaunchKernelGGL((embed_kernel<4, true>), grid4, dim3(256), 0, st, A);
            else hipLaunchKernelGGL((embed_kernel<4, false>), grid4, dim3(256), 0, st, A);
        }
    } else if (h->d.kind == 0 && A.P == 4 && A.Cin == 3) hipLaunchKernelGGL((downsample_kernel<0, 4, 3>), grid, dim3(256), lds, st, A);
    else if (h->d.kind == 0) hipLaunchKernelGGL(downsample_kernel<0>, grid, dim3(256), lds, st, A);
    else hipLaunchKernelGGL(downsample_kernel<1>, grid, dim3(256), lds, st, A);
    HIP_TRY(hipGetLastError());
    return MIXAQ_OK;
}

}  // namespace

extern "C" {

int mixaq_downsample_out_shape(const mixaq_downsample_desc* desc, int32_t* Ho, int32_t* Wo, int32_t* K)
{
    if (!Ho || !Wo || !K) return fail(MIXAQ_E_NULL, "an output pointer is NULL");
    int P, k, ho, wo, rc = ds_geometry(desc, &P, &k, &ho, &wo);
    if (rc) return rc;
    *Ho = ho; *Wo = wo; *K = k;
    return MIXAQ_OK;
}

static int downsample_create(const mixaq_downsample_desc* desc, const mixaq_downsample_params* p, mixaq_downsample** out);

// No C++ exception leaves the library: host containers that fail to allocate become an error code.
int mixaq_downsample_create(const mixaq_downsample_desc* desc, const mixaq_downsample_params* p, mixaq_downsample** out)
{
    try {
        return downsample_create(desc, p, out);
    } catch (const std::bad_alloc&) {
        return fail(MIXAQ_E_HIP, "out of host memory while preparing the layer");
    } catch (...) {
        return fail(MIXAQ_E_HIP, "unexpected C++ exception while preparing the layer");
    }
}

namespace {
struct LayerOwner {                      // frees a half-built layer on every early return and on an exception
    mixaq_downsample* h;
    ~LayerOwner() { delete h; }
};
}  // namespace

static int downsample_create(const mixaq_downsample_desc* desc, const mixaq_downsample_params* p, mixaq_downsample** out)
{
    if (!out) return fail(MIXAQ_E_NULL, "out is NULL");
    *out = nullptr;
    int P, K, Ho, Wo, rc = ds_geometry(desc, &P, &K, &Ho, &Wo);
    if (rc) return rc;
    if (!p || !p->w || !p->s_w || !p->ln_gamma || !p->ln_beta) return fail(MIXAQ_E_NULL, "a required parameter pointer is NULL");
    if (!(p->a_in.scale > 0.0f) || !std::isfinite(p->a_in.scale)) return fail(MIXAQ_E_SHAPE, "input scale must be positive");
    const int qmin = -(1 << (desc->act_bits - 1)), qmax = (1 << (desc->act_bits - 1)) - 1;
    if (p->a_in.zero_point < qmin || p->a_in.zero_point > qmax) return fail(MIXAQ_E_BITS, "zero point outside the code range");
    const int N = desc->N, Kp = (K + 31) / 32 * 32, n_ln = desc->kind == 0 ? N : K;
    if (desc->kind == 0 && (size_t)Kp * 32 + (size_t)32 * N * 4 > 64 * 1024) return fail(MIXAQ_E_SHAPE, "patch embedding too wide for one workgroup's LDS");
    if ((size_t)Kp * 32 > 64 * 1024) return fail(MIXAQ_E_SHAPE, "too many inputs per token for one workgroup's LDS");
    mixaq_downsample* h = new (std::nothrow) mixaq_downsample();
    if (!h) return fail(MIXAQ_E_HIP, "out of host memory");
    LayerOwner owner{h};
    auto bail = [&](int code) { return code; };          // the owner frees the layer
    h->d = *desc; h->P = P; h->K = K; h->Kp = Kp; h->Ho = Ho; h->Wo = Wo;
    h->by_map = FastDiv(Ho * Wo); h->by_row = FastDiv(Wo);
    std::vector<int8_t> w((size_t)N * K);
    std::vector<float> s(N), bias(N, 0.0f), ln_g(n_ln), ln_b(n_ln);
    if (hipMemcpy(w.data(), p->w, w.size(), hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemcpy(s.data(), p->s_w, (size_t)N * 4, hipMemcpyDeviceToHost) != hipSuccess ||
        (p->bias && hipMemcpy(bias.data(), p->bias, (size_t)N * 4, hipMemcpyDeviceToHost) != hipSuccess) ||
        hipMemcpy(ln_g.data(), p->ln_gamma, (size_t)n_ln * 4, hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemcpy(ln_b.data(), p->ln_beta, (size_t)n_ln * 4, hipMemcpyDeviceToHost) != hipSuccess)
        return bail(fail(MIXAQ_E_HIP, "copy of the parameters to the host failed"));
    const int wmax = (1 << (desc->weight_bits - 1)) - 1, wmin = -(1 << (desc->weight_bits - 1));
    std::vector<float> m(N);
    std::vector<int> nc(N);
    for (int n = 0; n < N; ++n) {
        if (!(s[n] > 0.0f) || !std::isfinite(s[n])) return bail(fail(MIXAQ_E_SHAPE, "weight scale %d is not positive", n));
        long long cs = 0;
        for (int k = 0; k < K; ++k) {
            const int v = w[(size_t)n * K + k];
            if (v < wmin || v > wmax) return bail(fail(MIXAQ_E_BITS, "weight code %d outside the %d-bit range", v, desc->weight_bits));
            cs += v;
        }
        m[n] = p->a_in.scale * s[n];
        nc[n] = (int)(-(long long)p->a_in.zero_point * cs);
    }
    const int NB = N / 32, KS = Kp / 32;
    const bool halves = embed_in_registers(*desc);
    std::vector<int8_t> packed((size_t)N * Kp, 0);
    for (int nb = 0; nb < NB; ++nb)
        for (int ks = 0; ks < KS; ++ks)
            for (int lane = 0; lane < 64; ++lane)
                for (int e = 0; e < 16; ++e) {
                    // of the halves: 16 k each per slab, or 24 each in all (embed_kernel)
                    const int k = !halves ? ks * 32 + (lane / 32) * 16 + e : ks * 16 + e < K / 2 ? (lane / 32) * (K / 2) + ks * 16 + e : K;
                    if (k < K) packed[(((size_t)nb * KS + ks) * 64 + lane) * 16 + e] = w[(size_t)(nb * 32 + lane % 32) * K + k];
                }
    h->mem.add(packed, &h->Wp);
    h->mem.add(m, &h->m);
    h->mem.add(bias, &h->bias);
    h->mem.add(nc, &h->negcorr);
    h->mem.add(ln_g, &h->gamma);
    h->mem.add(ln_b, &h->beta);
    HIP_TRY(h->mem.commit());
    h->q.scale = p->a_in.scale;
    h->q.zp = p->a_in.zero_point;
    h->q.inv_s = 1.0f / p->a_in.scale;
    h->q.magic = RND_MAGIC + (float)p->a_in.zero_point;
    h->q.lo = RND_MAGIC + (float)qmin;
    h->q.hi = RND_MAGIC + (float)qmax;
    owner.h = nullptr;
    *out = h;
    return MIXAQ_OK;
}

int mixaq_downsample_destroy(mixaq_downsample* h)
{
    delete h;
    return MIXAQ_OK;
}

int mixaq_downsample_forward(const mixaq_downsample* h, const float* x, float* y, void* stream)
{
    return ds_forward(h, x, y, stream, nullptr, nullptr);
}

int mixaq_downsample_forward_taps(const mixaq_downsample* h, const float* x, float* y, void* stream, int8_t* tap_codes,
                                  int32_t* tap_acc)
{
    return ds_forward(h, x, y, stream, tap_codes, tap_acc);
}

}  // extern "C"
