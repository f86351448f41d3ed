// gfx950 kernels of the Two-Branch Swin Block (paper Sec. 3.2, Fig. 3):
//   score_kernel      window importance = squared L2 norm            (Sec. 3.2)
//   select_rank_kernel  top-k partition into high / low groups       (Sec. 3.2)
//   window_kernel     gather + LN1 + QKV + attention of a window; wide blocks take LN1 from ln_window_kernel
//   token_kernel      projection + LN2 + FFN + scatter of a tile of rows
//   block_kernel      both of them for a window, on few windows
// and, where these do not apply,
//   ln_quant_kernel   gather (shift folded in) + LayerNorm + quantize, also LN2
//   gemm_ring_kernel, gemm_few_kernel, gemm_tile_kernel  int8 MFMA linear layers with fused epilogues (shadow layers): long K, long K on
//                     few rows, short or odd K
//   attn_kernel       per (window, head): QK^T, bias+mask, softmax, P.V
// Arithmetic that decides an integer code follows the pinned binary32 sequences
// of mixaq_dev.h; reductions feeding a code run in binary64.
#include <algorithm>
#include <type_traits>
#include "mixaq_dev.h"
#include "kernels.h"

namespace mixaq {

// ------------------------------------------------------------------ helpers
// sum over a group of W consecutive lanes (the group does not straddle a wave; first = its first lane); every lane of the
// group gets the same bits: a butterfly for powers of two; otherwise W = 3 * 2^k, a butterfly over the aligned subgroups of
// 2^k lanes, then three shuffles (over all W lanes they were 24 permutes through the LDS pipe and eleven dependent additions at
// W = 12).
template <int W>
__device__ __forceinline__ double group_sum(double v, int first = 0)
{
    if constexpr ((W & (W - 1)) == 0) return lanes_sum<W>(v);
    else {
        constexpr int P = W & -W;
        static_assert(W == 3 * P && P <= 4, "three aligned subgroups of one quad at most");
        v = lanes_sum<P>(v);
        return (__shfl(v, first, 64) + __shfl(v, first + P, 64)) + __shfl(v, first + 2 * P, 64);
    }
}

// LayerNorm of one token spread over LPT lanes (NV float4 per lane; channel of
// element e of vector k on lane i: (k*LPT + i)*4 + e).  Mean and variance in
// binary64, rounded once (see ln_stats.h).
template <int LPT, int NV>
__device__ __forceinline__ void token_ln_stats(float4 (&v)[NV], int C, float eps, float& mean, float& rstd, int first = 0)
{
    double s = 0.0, q = 0.0;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        if (NV > 8 && k % 4 == 0) __builtin_amdgcn_sched_barrier(0);
        s += sum4(v[k].x, v[k].y, v[k].z, v[k].w);
    }
    mean = ln_mean(group_sum<LPT>(s, first), C);
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        if (NV > 8 && k % 4 == 0) __builtin_amdgcn_sched_barrier(0);
        q += centred4<true>(v[k].x, v[k].y, v[k].z, v[k].w, mean);
    }
    rstd = ln_rstd(group_sum<LPT>(q, first), C, eps);
}

template <int LPT, int NV>
__device__ __forceinline__ void token_ln_apply(float4 (&v)[NV], float mean, float rstd, const float* __restrict__ gamma,
                                               const float* __restrict__ beta, int sub)
{
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        if (NV > 8 && k % 4 == 0) __builtin_amdgcn_sched_barrier(0);     // long tokens: a few parameter reads in flight, not all of them
        int ch = (k * LPT + sub) * 4;
        float4 g = *(const float4*)(gamma + ch), b = *(const float4*)(beta + ch);
        v[k].x = fmaf((v[k].x - mean) * rstd, g.x, b.x);
        v[k].y = fmaf((v[k].y - mean) * rstd, g.y, b.y);
        v[k].z = fmaf((v[k].z - mean) * rstd, g.z, b.z);
        v[k].w = fmaf((v[k].w - mean) * rstd, g.w, b.w);
    }
}

// the same with gamma and beta requested ahead (a kernel that is one chain of waits: the parameters travel with the token)
template <int NV> struct Affine { float4 g[NV], b[NV]; };
template <int LPT, int NV>
__device__ __forceinline__ void request_affine(Affine<NV>& a, const float* __restrict__ gamma, const float* __restrict__ beta, int sub)
{
#pragma unroll
    for (int k = 0; k < NV; ++k) { a.g[k] = *(const float4*)(gamma + (k * LPT + sub) * 4); a.b[k] = *(const float4*)(beta + (k * LPT + sub) * 4); }
}
template <int LPT, int NV>
__device__ __forceinline__ void token_layernorm(float4 (&v)[NV], int C, float eps, const Affine<NV>& a)
{
    float mean, rstd;
    token_ln_stats<LPT, NV>(v, C, eps, mean, rstd);
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        v[k].x = fmaf((v[k].x - mean) * rstd, a.g[k].x, a.b[k].x);
        v[k].y = fmaf((v[k].y - mean) * rstd, a.g[k].y, a.b[k].y);
        v[k].z = fmaf((v[k].z - mean) * rstd, a.g[k].z, a.b[k].z);
        v[k].w = fmaf((v[k].w - mean) * rstd, a.g[k].w, a.b[k].w);
    }
}

template <int LPT, int NV>
__device__ __forceinline__ void token_layernorm(float4 (&v)[NV], int C, float eps, const float* __restrict__ gamma,
                                                const float* __restrict__ beta, int sub, int first = 0)
{
    float mean, rstd;
    token_ln_stats<LPT, NV>(v, C, eps, mean, rstd, first);
    token_ln_apply<LPT, NV>(v, mean, rstd, gamma, beta, sub);
}

// ------------------------------------------------------------------ K0 score
// One workgroup of NT threads per window of the un-shifted grid, LPT lanes per token.  The loads of PC passes over the
// tokens are issued together, before any arithmetic.  Memory bound once there are windows enough to fill the chip; wide maps
// have few windows, each of them a chain of round trips for its one workgroup, so from C = 384 it gets 1024 threads that have
// the whole window in flight at once (see launch_score_t).
template <int LPT, int NV, int NT>
__global__ __launch_bounds__(NT) void score_kernel(Geom G, const float* __restrict__ x, int mode, float eps,
                                                   const float* __restrict__ gamma, const float* __restrict__ beta,
                                                   double* __restrict__ scores)
{
    const int wid = blockIdx.x;                       // b*nW + w
    const int b = G.by_nW(wid), w = wid - b * G.nW;
    const int wr = G.by_nWc(w), wc = w - wr * G.nWc;
    const int grp = threadIdx.x / LPT, sub = threadIdx.x % LPT;
    constexpr int TP = NT / LPT;
    double acc = 0.0;
    constexpr int PASSES = (TOK + TP - 1) / TP;
    constexpr int PC = LPT <= 16 || NT > 256 ? PASSES : 2;
#pragma unroll 1
    for (int p0 = 0; p0 < PASSES; p0 += PC) {
        float4 v[PC][NV];
        bool in[PC];
#pragma unroll
        for (int p = 0; p < PC; ++p) {
            const int t = grp + (p0 + p) * TP, pr = wr * WS + t / WS, pc = wc * WS + t % WS;
            in[p] = t < TOK && pr < G.H && pc < G.W;  // uniform inside a token group
            if (in[p]) {
                const float* px = x + ((size_t)(b * G.H + pr) * G.W + pc) * (LPT * NV * 4);
#pragma unroll
                for (int k = 0; k < NV; ++k) v[p][k] = *(const float4*)(px + (k * LPT + sub) * 4);
            }
        }
#pragma unroll
        for (int p = 0; p < PC; ++p) {
            if (in[p]) {
                if (mode == 1) token_layernorm<LPT, NV>(v[p], LPT * NV * 4, eps, gamma, beta, sub);
#pragma unroll
                for (int k = 0; k < NV; ++k) {
                    const double d0 = v[p][k].x, d1 = v[p][k].y, d2 = v[p][k].z, d3 = v[p][k].w;
                    acc += __builtin_fma(d0, d0, d1 * d1) + __builtin_fma(d2, d2, d3 * d3);
                }
            }
        }
    }
    acc = group_sum<64>(acc);
    __shared__ double part[NT / 64];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < NT / 64; ++k) s += part[k];
        scores[wid] = s;
    }
}

// ------------------------------------------------------------------ K1 select
// Rank by counting under the total order (score descending, index ascending): the rank of a
// window is the number of windows ahead of it, which is a permutation, so perm[rank] = window
// lists the windows by decreasing importance; the high group is the first k_hi entries.
// A wave ranks four windows at once, its lanes stride over the candidates held in LDS.
// A score that is not a number (a window holding NaN, or Inf under the scoring LayerNorm) is outside
// the order: it is ranked behind every number (infinities included), so the ranks stay a permutation.
// rank_key maps it to the infinity at the unimportant end; among equal keys a number goes first.
__device__ __forceinline__ double rank_key(double s, int reverse)
{
    const double worst = reverse ? __longlong_as_double(0x7ff0000000000000LL) : __longlong_as_double(0xfff0000000000000LL);
    return s != s ? worst : s;
}
// true when candidate v (raw score rv) is ranked before window w (raw score rw)
__device__ __forceinline__ bool ranked_before(double rv, int v, double rw, int w, int reverse)
{
    const double sv = rank_key(rv, reverse), sw = rank_key(rw, reverse);
    const bool nv = rv != rv, nw = rw != rw;
    const bool ahead = reverse ? (sv < sw) : (sv > sw);
    return ahead || (sv == sw && (nv != nw ? nw : v < w));
}
// Rank of window w of an image: how many of its windows come before it (order of importance).  The whole workgroup of NT
// threads takes part and gets the same number; red: one int per wave, LDS.  Counted by ballot: four vector instructions per
// candidate (the sorted order needs the NaN rules of ranked_before only when w's own score is NaN: a NaN candidate compares
// false both ways, which ranks it behind every number).
template <int NT>
__device__ __forceinline__ int window_rank(const double* __restrict__ sc, int nW, int w, int tid, int* red)
{
    const double sw = sc[w];
    int cnt = 0;
    for (int base = 0; base < nW; base += 8 * NT) {                      // eight loads in flight per thread
        double sv[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) sv[k] = sc[min(base + tid + k * NT, nW - 1)];
        if (sw == sw) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int u = base + tid + k * NT;
                cnt += __popcll(__ballot(u < nW && (sv[k] > sw || (sv[k] == sw && u < w))));
            }
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int u = base + tid + k * NT;
                cnt += __popcll(__ballot(u < nW && ranked_before(sv[k], u, sw, w, 0)));
            }
        }
    }
    if ((tid & 63) == 0) red[tid >> 6] = cnt;
    __syncthreads();
    int rank = 0;
#pragma unroll
    for (int k = 0; k < NT / 64; ++k) rank += red[k];
    return __builtin_amdgcn_readfirstlane(rank);                          // the same in every lane: what follows from it stays scalar
}
constexpr int RANK_WPB = 16;                          // windows ranked per workgroup (4 per wave)
__global__ __launch_bounds__(256) void select_rank_kernel(const double* __restrict__ scores, int nW, int reverse,
                                                          int* __restrict__ perm)
{
    extern __shared__ double rsc[];                   // all scores of the image
    const int b = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const double* sc = scores + (size_t)b * nW;
    for (int base = 0; base < nW; base += 2048) {     // eight loads in flight per thread
        double tmp[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) { const int i = base + threadIdx.x + k * 256; tmp[k] = i < nW ? sc[i] : 0.0; }
#pragma unroll
        for (int k = 0; k < 8; ++k) { const int i = base + threadIdx.x + k * 256; if (i < nW) rsc[i] = tmp[k]; }
    }
    __syncthreads();
    constexpr int Q = RANK_WPB / 4;                   // windows per wave, ranked together
    const int w0 = blockIdx.x * RANK_WPB + wave * Q;
    if (w0 >= nW) return;                             // whole wave, after the barrier
    double sw[Q];
    int rank[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) { sw[q] = rsc[min(w0 + q, nW - 1)]; rank[q] = 0; }
    for (int v0 = lane; v0 < nW; v0 += 256) {
        double sv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) { const int v = v0 + 64 * u; sv[u] = rsc[min(v, nW - 1)]; }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int v = v0 + 64 * u;
#pragma unroll
            for (int q = 0; q < Q; ++q) rank[q] += (v < nW && ranked_before(sv[u], v, sw[q], w0 + q, reverse)) ? 1 : 0;
        }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) rank[q] += __shfl_xor(rank[q], o, 64);
        if (lane == 0 && w0 + q < nW) perm[(size_t)b * nW + rank[q]] = w0 + q;
    }
}

// ------------------------------------------------------------------ pruned windows
// Activation pruning (paper Sec. 3.4): the windows after the high and low groups in perm are
// skipped by the block and their features are forwarded.  One workgroup per pruned window.
__global__ __launch_bounds__(256) void bypass_kernel(Geom G, const int* __restrict__ perm, const float* __restrict__ x,
                                                     float* __restrict__ y)
{
    const int kept = G.k_hi + G.k_lo, n_pruned = G.nW - kept;
    const int b = blockIdx.x / n_pruned, jpos = kept + blockIdx.x % n_pruned;
    const int w = perm[b * G.nW + jpos];
    const int wr = G.by_nWc(w), wc = w - wr * G.nWc;
    const int c4 = G.C / 4;
    for (int i = threadIdx.x; i < TOK * c4; i += 256) {
        const int t = i / c4, k = i - t * c4, tr = t / WS, tc = t - tr * WS;
        int pr = wr * WS + tr + G.shift; if (pr >= G.Hp) pr -= G.Hp;
        int pc = wc * WS + tc + G.shift; if (pc >= G.Wp) pc -= G.Wp;
        if (pr < G.H && pc < G.W) {
            const size_t off = ((size_t)(b * G.H + pr) * G.W + pc) * G.C + k * 4;
            *(float4*)(y + off) = *(const float4*)(x + off);
        }
    }
}

// ------------------------------------------------------------------ K2 / K6
// One token per group of LPT lanes.  GATHER: source is the feature map through the
// window / shift / padding index map, and the row bookkeeping is written.
template <int LPT, int NV, bool GATHER>
__global__ __launch_bounds__(256) void ln_quant_kernel(Geom G, LnArgs A)
{
    touch_arguments<sizeof(Geom) + sizeof(LnArgs)>();
    constexpr int TP = 256 / LPT;
    const int row = blockIdx.x * TP + threadIdx.x / LPT, sub = threadIdx.x % LPT;
    if (row >= G.rows_total) return;
    int branch, canon, pix;
    float4 v[NV];
    if (GATHER) {
        RowInfo ri = row_info(G, A.perm, row);
        branch = ri.branch; canon = ri.canon; pix = ri.pix;
        if (sub == 0) { A.row_pix[row] = pix; A.row_canon[row] = canon; }
    } else {
        branch = row >= G.base_lo ? 1 : 0;
        canon = A.row_canon[row];
        pix = 0;
    }
    const QDev q = in_vgpr(A.q[branch]);
    // h and the parameters with the row's mark, not behind it: every row of the region has its place in h (16 windows
    // at C = 512, six blocks 242.6 -> 240.4 us; the kernel itself on 24 windows at C = 768 4.8 -> 3.7)
    Affine<NV> af;
    const float* src = A.src + (GATHER ? (size_t)max(pix, 0) : (size_t)row) * G.C;
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = *(const float4*)(src + (k * LPT + sub) * 4);
    request_affine<LPT, NV>(af, A.gamma[branch], A.beta[branch], sub);
    if (canon >= 0 && pix >= 0) {
        token_layernorm<LPT, NV>(v, LPT * NV * 4, A.eps, af);
    } else {
#pragma unroll
        for (int k = 0; k < NV; ++k) v[k] = make_float4(0.f, 0.f, 0.f, 0.f);   // padding enters as LN output 0
    }
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        int code = pack4(quant_code(v[k].x, q), quant_code(v[k].y, q), quant_code(v[k].z, q), quant_code(v[k].w, q));
        if (canon < 0) code = 0;
        int ch = (k * LPT + sub) * 4;
        *(int*)(A.out + (GATHER ? frag_offset(row, ch, G.C / 32) : frag_offset_reg(row, ch, G.C / 32))) = code;   // the k order of the next layer's weights
        if (A.tap && canon >= 0) *(int*)(A.tap + (size_t)canon * G.C + ch) = code;
    }
}

// ------------------------------------------------------------------ GEMMs
// out^T = W * act^T on 32x32x32 int8 MFMA: the packed weight fragment is the A
// operand (rows = output channels), the activation rows are the B operand (columns
// = tokens), so a lane owns one token and 16 output channels per 32-channel block.
// A wave computes 64 rows x 32 channels at a time.
// What the epilogue of one 32-channel block reads besides the sums; requested before the block's chain of products, so
// that it travels under it.
struct EpiConst { float4 m[4], bias[4]; };
template <int EPI>
__device__ __forceinline__ void epilogue_residual(const GemmArgs& A, int row, int nb, int g, int pix, float4 (&res)[4])
{
#pragma unroll
    for (int qd = 0; qd < 4; ++qd) {
        const int n0 = nb * 32 + qd * 8 + g * 4;
        if (EPI == EPI_PROJ) res[qd] = pix >= 0 ? *(const float4*)(A.x + (size_t)pix * A.N + n0) : make_float4(0.f, 0.f, 0.f, 0.f);
        if (EPI == EPI_FC2) res[qd] = *(const float4*)(A.resid + (size_t)row * A.N + n0);
    }
}
template <int EPI, bool STEPS = false>
__device__ __forceinline__ void epilogue(const GemmArgs& A, const Geom& G, int branch, int row, int nb, int g, const v16i& acc,
                                         const EpiConst& ec, const float4 (&res)[4], int pix, int canon, const float4* gelu_lds)
{
    const int N = A.N;
    int codes[4];
#pragma unroll
    for (int qd = 0; qd < 4; ++qd) {
        const int n0 = nb * 32 + qd * 8 + g * 4;
        const float4 m = ec.m[qd], bs = ec.bias[qd];
        const int a0 = acc[qd * 4 + 0], a1 = acc[qd * 4 + 1], a2 = acc[qd * 4 + 2], a3 = acc[qd * 4 + 3];
        const float f0 = fmaf((float)a0, m.x, bs.x), f1 = fmaf((float)a1, m.y, bs.y);
        const float f2 = fmaf((float)a2, m.z, bs.z), f3 = fmaf((float)a3, m.w, bs.w);
        if (A.tap_acc && canon >= 0) *(int4*)(A.tap_acc + (size_t)canon * N + n0) = make_int4(a0, a1, a2, a3);
        if (EPI == EPI_QKV || EPI == EPI_FC1) {
            const QDev& q = A.q[branch][EPI == EPI_QKV ? n0 / G.C : 0];
            if (EPI == EPI_FC1 && STEPS) {
                GeluStepPart p = {{f0, f1, f2, f3}, {}};
                gelu_begin(p, (const GeluStep*)gelu_lds, in_vgpr(A.step_index[branch]));
                codes[qd] = gelu_end(p);
            } else if (EPI == EPI_FC1) {
                GeluPart p = {{f0, f1, f2, f3}, {}, {}};
                gelu_begin(p, gelu_lds);
                codes[qd] = gelu_end(p, q);
            } else codes[qd] = pack4(quant_code(f0, q), quant_code(f1, q), quant_code(f2, q), quant_code(f3, q));
            if (EPI == EPI_QKV) *(int*)(A.out8 + (size_t)row * N + n0) = codes[qd];
            if (A.tap_code && canon >= 0) *(int*)(A.tap_code + (size_t)canon * N + n0) = codes[qd];
        } else {   // PROJ: first residual (the shortcut); FC2: second residual and scatter back to the map
            const float4 o = make_float4(f0 + res[qd].x, f1 + res[qd].y, f2 + res[qd].z, f3 + res[qd].w);
            if (EPI == EPI_PROJ) *(float4*)(A.outf + (size_t)row * N + n0) = o;
            else if (pix >= 0) *(float4*)(A.y + (size_t)pix * N + n0) = o;
            if (A.tap_f && canon >= 0) *(float4*)(A.tap_f + (size_t)canon * N + n0) = o;
        }
    }
    // FC1: the lane's 16 codes are one lane's 16 bytes of FC2's operand fragment (k in the order of the result registers)
    if (EPI == EPI_FC1) *(v4i*)(A.out8 + (((size_t)(row >> 5) * (N / 32) + nb) * 64 + g * 32 + (row & 31)) * 16) = (v4i){codes[0], codes[1], codes[2], codes[3]};
}

// One workgroup per tile of RT rows and group of output blocks (all of them once the tiles alone fill the chip).  For what the
// other two do not take (see product_form): K below 512 or no multiple of 128, or N no multiple of 64; the longest K is 1344.  The activations
// come as MFMA operand fragments ([32 rows][K slab][64 lanes][16 bytes], written so by their producers), so a tile is a contiguous run of
// memory: it goes to LDS by direct loads, no register in between, all of them in flight together.  Wave w computes the
// output blocks first + w, first + w + 4, ... of the group; its weight fragments stream through a ring of D loads that
// starts before anything else and runs on across the output blocks.
// KMAX: bytes of K the instantiation's LDS holds per row
template <int EPI, int KMAX, int RT, int D>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(RT * KMAX <= 65536 ? 2 : 1))) void gemm_tile_kernel(Geom G, GemmArgs A)
{
    touch_arguments<sizeof(Geom) + sizeof(GemmArgs)>();
    constexpr int RB = RT / 32, PF = D % 4 == 0 ? 4 : 3;                // PF: LDS reads ahead
    static_assert(D % PF == 0, "the LDS slots come round with the ring");
    __shared__ v4i afr[RT * KMAX / 16];                                // [row blocks][slabs][64 lanes]
    __shared__ float4 gtab[EPI == EPI_FC1 ? GELU_K : 1];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, j = lane & 31, g = lane >> 5;
    const int row0 = blockIdx.x * RT;
    const int branch = row0 >= G.base_lo ? 1 : 0;
    const int K = A.K, ks_n = K / 32, NB = A.N / 32;
    const int nb_lo = blockIdx.y * A.nb_per_block, nb_hi = min(nb_lo + A.nb_per_block, NB);
    const v4i* wp = A.Wp + (size_t)min(nb_lo + wave, NB - 1) * ks_n * 64 + lane;
    int pix[RB], canon[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        canon[rb] = A.row_canon[row0 + rb * 32 + j];
        pix[rb] = (EPI == EPI_PROJ || EPI == EPI_FC2) ? A.row_pix[row0 + rb * 32 + j] : 0;
    }
    v4i rw[D];
#pragma unroll
    for (int d = 0; d < D; ++d) rw[d] = wp[min(d, ks_n - 1) * 64];     // K may hold fewer than D slabs: the last one again (unused)
    for (int f = wave; f < RB * ks_n; f += 4) {                        // one fragment of the tile per wave and turn; the whole K stays for every output block
        const int rb = f >= ks_n ? 1 : 0;
        const int8_t* src = A.A + ((size_t)(blockIdx.x * RB + rb) * ks_n + f - rb * ks_n) * 1024 + lane * 16;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                         (__attribute__((address_space(3))) void*)(afr + f * 64), 16, 0, 0);
    }
    // what a block's start and epilogue read, requested ahead of its products (for the first block: with the tile)
    int4 nc[4];
    EpiConst ec;
    float4 res[RB][4];
    auto request = [&](int nb) {
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
            const int n0 = nb * 32 + qd * 8 + g * 4;
            nc[qd] = *(const int4*)(A.negcorr[branch] + n0);
            ec.m[qd] = *(const float4*)(A.m[branch] + n0);
            ec.bias[qd] = *(const float4*)(A.bias[branch] + n0);
        }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) epilogue_residual<EPI>(A, row0 + rb * 32 + j, nb, g, pix[rb], res[rb]);
    };
    request(min(nb_lo + wave, NB - 1));
    if (EPI == EPI_FC1) gelu_stage_table(gtab, A.gelu_tab, tid, 256);
    const float4* gelu_lds = gtab;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                   // the direct loads have landed
    __syncthreads();
    for (int nb0 = nb_lo; nb0 < nb_hi; nb0 += 4) {                     // the same trips for every wave: barriers inside
        const int nb = min(nb0 + wave, NB - 1);
        const bool active = nb0 + wave < nb_hi;
        const v4i* wnext = A.Wp + (size_t)min(nb0 + 4 + wave, NB - 1) * ks_n * 64 + lane;
        if (nb0 > nb_lo) request(nb);
        v16i c0, c1;                                                     // c1: the second row block (RT = 64)
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {                                 // accumulators start at -zp_in * colsum(W[n,:])
            c0[qd * 4 + 0] = nc[qd].x; c0[qd * 4 + 1] = nc[qd].y; c0[qd * 4 + 2] = nc[qd].z; c0[qd * 4 + 3] = nc[qd].w;
        }
        c1 = c0;
        // One turn of the ring: D fragments are used, the D after them requested.  Every step is product, request into
        // the slot just used, next LDS read, in this order: left free, the scheduler moves the requests up, the slots of
        // the next turn need registers of their own, and the copies at the turn's end wait for every load in flight.
        v4i b[PF][RB];
#pragma unroll
        for (int d = 0; d < PF; ++d)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) b[d][rb] = afr[(rb * ks_n + min(d, ks_n - 1)) * 64 + lane];
        auto turn = [&](int k0, auto full) {
            const bool last = k0 + D >= ks_n;                            // the ring turns to the next output block's weights
            const v4i* wsrc = last ? wnext : wp + (size_t)(k0 + D) * 64;
            const int left = last ? ks_n - 1 : ks_n - 1 - (k0 + D);
#pragma unroll
            for (int d = 0; d < D; ++d) {
                if (decltype(full)::value || k0 + d < ks_n) {            // wave-uniform: the last turn may be partial
                    c0 = mfma32(rw[d], b[d % PF][0], c0);
                    if (RB == 2) c1 = mfma32(rw[d], b[d % PF][RB - 1], c1);
                }
                rw[d] = wsrc[min(d, left) * 64];                         // past the end: the last slab again (unused)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) b[d % PF][rb] = afr[(rb * ks_n + min(k0 + d + PF, ks_n - 1)) * 64 + lane];
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        int k0 = 0;
#pragma unroll 1
        for (; k0 + D <= ks_n; k0 += D) turn(k0, std::true_type());
        if (k0 < ks_n) turn(k0, std::false_type());
        wp = wnext;
        if (active) {
            epilogue<EPI>(A, G, branch, row0 + j, nb, g, c0, ec, res[0], pix[0], canon[0], gelu_lds);
            if (RB == 2) epilogue<EPI>(A, G, branch, row0 + 32 + j, nb, g, c1, ec, res[RB - 1], pix[RB - 1], canon[RB - 1], gelu_lds);
        }
    }
}

// The same products for many rows: both operands through LDS.  A workgroup computes RT = 32 WY RB rows times NT = 32 WX NBW
// channels, wave (wy, wx) the RB x NBW blocks of its corner, so that an operand fragment read from LDS feeds RB or NBW products
// instead of one or two, and a byte from the caches RT or NT of them: see product_form for the times.  K passes in stages of KSL slabs through a ring
// of S LDS buffers filled by direct loads; a stage is requested S - 1 stages ahead, into the buffer that all waves have left at the barrier
// in front of it, and that barrier is the only one of a stage.  The residual is requested ahead of the last S - 2 stages and travels under
// their products, a further tile's first stages ahead of the epilogue: they travel under FC1's.  In the projection's and FC2's the residual's quads are
// awaited one by one between stores that the compiler cannot count (each depends on a tap or a pixel) and behind loads it does not know of;
// the counter goes down in order, so from the second quad on a wait includes the tile's own earlier stores, and the last one those stages too.
// What bounds it: on many rows the epilogue's memory (the projection on 19 712 rows at C = 768 33 us, of them 26 its maps at the rate of a
// copy; without any epilogue 14) and the GELU; on few, the ramp of launch, first loads and the chain of stages.
// The direct loads are asm: as a builtin every LDS read behind them waits for all of them.
template <int N>
__device__ __forceinline__ void request_to_lds(const void* uniform_src, int lane_bytes, unsigned lds_dst)
{
    static_assert(N == 1 || N == 2 || N == 4, "written out for these");
    int m0;                                                              // given back: the compiler does not let an asm statement change it
#define MIXAQ_REQUEST(MORE_) \
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3\n\t" MORE_ "s_mov_b32 m0, %0" \
                 : "=&s"(m0) : "s"(lds_dst), "v"(lane_bytes), "s"(uniform_src) : "memory")
    if constexpr (N == 1) MIXAQ_REQUEST("");
    if constexpr (N == 2) MIXAQ_REQUEST("global_load_lds_dwordx4 %2, %3 offset:1024\n\t");
    if constexpr (N == 4) MIXAQ_REQUEST("global_load_lds_dwordx4 %2, %3 offset:1024\n\tglobal_load_lds_dwordx4 %2, %3 offset:2048\n\tglobal_load_lds_dwordx4 %2, %3 offset:3072\n\t");
#undef MIXAQ_REQUEST
}
__device__ __forceinline__ void group_barrier() { asm volatile("" ::: "memory"); __builtin_amdgcn_s_barrier(); asm volatile("" ::: "memory"); }
template <int N> __device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(N) : "memory"); }
template <int EPI, int WY, int WX, int RB, int NBW, int KSL, int S, int WPE, bool STEPS>
__global__ __launch_bounds__(WY * WX * 64) __attribute__((amdgpu_waves_per_eu(WPE))) void gemm_ring_kernel(Geom G, GemmArgs A)
{
    constexpr int W = WY * WX, AF = WY * RB * KSL, FR = AF + WX * NBW * KSL, LPW = FR / W, NT = WX * NBW * 32, RT = WY * RB * 32;
    constexpr int CST = (3 * NT + 255) / 256;                            // 1 KB pieces of a tile's constants
    static_assert(FR % W == 0 && S >= 3 && S <= 4 && LPW * (S - 2) < 64 && CST <= W, "whole fragments a wave; the counter of loads in flight");
    __shared__ v4i buf[S][FR * 64];
    __shared__ __attribute__((aligned(16))) float cst[2][3 * NT];        // [m | bias | negcorr] of a tile's channels, this tile's and the next one's
    __shared__ float4 gtab[EPI != EPI_FC1 ? 1 : STEPS ? GELU_STEP_PIECES * 64 : GELU_K];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, j = lane & 31, g = lane >> 5;
    const int wy = wave / WX, wx = wave % WX;
    // consecutive tiles (all channels of a run of rows) on one XCD, whose L2 then reads the rows once
    const int tiles_n = A.N / NT, tiles = (G.rows_total / RT) * tiles_n, per_xcd = (tiles + 7) / 8, step = gridDim.x / 8;
    const int last = min((int)(blockIdx.x & 7) * per_xcd + per_xcd, tiles);
    int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile >= last) return;                                            // the whole workgroup
    const int ks_n = A.K / 32, stages = ks_n / KSL;
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)buf, lds1 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)cst;
    constexpr int US = LPW % KSL == 0 ? KSL : KSL % 2 == 0 && LPW % 2 == 0 ? 2 : 1, UNITS = LPW / US;   // this wave requests UNITS runs of US slabs
    const int8_t* src[UNITS];
    int at = 0;
    auto request = [&](int slot) {
#pragma unroll
        for (int i = 0; i < UNITS; ++i) request_to_lds<US>(src[i], at, lds0 + (slot * FR + wave * LPW + i * US) * 1024);
        at += KSL * 1024;
    };
    // requests a tile's constants and its first S - 1 stages
    auto begin = [&](int t, int par) {
        const int tm = t / tiles_n, tn = t - tm * tiles_n, br = tm * RT >= G.base_lo ? 1 : 0;
        const int w = wave * 256 + lane * 4, n = tn * NT + w % NT;
        if (w < 3 * NT) {
            const float* from = w < NT ? A.m[br] + n : w < 2 * NT ? A.bias[br] + n : (const float*)A.negcorr[br] + n;
            int m0;
            asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, off\n\ts_mov_b32 m0, %0" : "=&s"(m0) : "s"(__builtin_amdgcn_readfirstlane(lds1 + par * (12 * NT) + wave * 1024)), "v"(from) : "memory");
        }
#pragma unroll
        for (int i = 0; i < UNITS; ++i) {
            const int f = wave * LPW + i * US, r = f / KSL, s = f % KSL;
            src[i] = r < WY * RB ? A.A + ((size_t)(tm * (WY * RB) + r) * ks_n + s) * 1024 : (const int8_t*)A.Wp + ((size_t)(tn * (WX * NBW) + r - WY * RB) * ks_n + s) * 1024;
        }
        at = lane * 16;
#pragma unroll
        for (int k = 0; k < S - 1; ++k) request(k);
    };
    int branch = -1, par = 0;
    begin(tile, 0);
    for (; tile < last; tile += step, par ^= 1) {
        const int tm = tile / tiles_n, tn = tile - tm * tiles_n, row0 = tm * RT;
        int pix[RB], canon[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int row = row0 + (wy * RB + rb) * 32 + j;
            canon[rb] = A.row_canon[row];
            pix[rb] = (EPI == EPI_PROJ || EPI == EPI_FC2) ? A.row_pix[row] : 0;
        }
        if (branch != (row0 >= G.base_lo ? 1 : 0)) {                     // once or twice: the tiles of a workgroup go up
            branch = row0 >= G.base_lo ? 1 : 0;
            if (EPI == EPI_FC1) {
                group_barrier();                            // the other branch's table is no longer read
                const float4* from = STEPS ? (const float4*)A.steps[branch] : A.gelu_tab;
                const int entries = STEPS ? A.step_pieces[branch] * 64 : GELU_K;
                for (int e = tid; e < entries; e += W * 64) gtab[e] = from[e];
            }
        }
        v16i acc[RB][NBW];
        auto products = [&](int slot) {
            const v4i *a = buf[slot] + wy * RB * KSL * 64 + lane, *w = buf[slot] + (AF + wx * NBW * KSL) * 64 + lane;
#pragma unroll
            for (int s = 0; s < KSL; ++s) {
                v4i av[RB], wv[NBW];
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) av[rb] = a[(rb * KSL + s) * 64];
#pragma unroll
                for (int nb = 0; nb < NBW; ++nb) wv[nb] = w[(nb * KSL + s) * 64];
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int nb = 0; nb < NBW; ++nb) acc[rb][nb] = mfma32(wv[nb], av[rb], acc[rb][nb]);
            }
        };
        int slot = 0;
        auto turn = [&](bool more) {
            if (more) request(slot == 0 ? S - 1 : slot - 1);
            products(slot);
            slot = slot == S - 1 ? 0 : slot + 1;
        };
        auto landed = [&] {                                              // a stage has landed, for every wave
            wait_loads<(S - 2) * LPW>();
            group_barrier();
        };
        landed();
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb) {                               // accumulators start at -zp_in * colsum(W[n,:])
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {
                const int4 t4 = *(const int4*)(&cst[par][2 * NT + (wx * NBW + nb) * 32 + qd * 8 + g * 4]);
                acc[0][nb][qd * 4 + 0] = t4.x; acc[0][nb][qd * 4 + 1] = t4.y; acc[0][nb][qd * 4 + 2] = t4.z; acc[0][nb][qd * 4 + 3] = t4.w;
            }
#pragma unroll
            for (int rb = 1; rb < RB; ++rb) acc[rb][nb] = acc[0][nb];
        }
        turn(true);
#pragma unroll 1
        for (int k = 1; k < stages - (S - 2); ++k) { landed(); turn(k + S - 1 < stages); }
        wait_loads<0>();                                                 // the last S - 2 stages together
        group_barrier();
        float4 res[RB][NBW][4];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)                                  // travels under them
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) epilogue_residual<EPI>(A, row0 + (wy * RB + rb) * 32 + j, tn * (WX * NBW) + wx * NBW + nb, g, pix[rb], res[rb][nb]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < S - 2; ++k) turn(false);
        if (tile + step < last) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");           // this wave's reads of the ring have returned
            group_barrier();
            begin(tile + step, par ^ 1);                                 // ahead of the epilogue
        }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) {
                const int row = row0 + (wy * RB + rb) * 32 + j, blk = tn * (WX * NBW) + wx * NBW + nb;
                EpiConst ec;
#pragma unroll
                for (int qd = 0; qd < 4; ++qd) {
                    const int n = (wx * NBW + nb) * 32 + qd * 8 + g * 4;
                    ec.m[qd] = *(const float4*)(&cst[par][n]);
                    ec.bias[qd] = *(const float4*)(&cst[par][NT + n]);
                }
                epilogue<EPI, STEPS>(A, G, branch, row, blk, g, acc[rb][nb], ec, res[rb][nb], pix[rb], canon[rb], gtab);
            }
    }
}

// The same products for few rows: one workgroup of eight waves per 32 x 32 outputs, each wave every eighth slab of K, SPW of them, its operands
// straight from memory to registers, as many requested at once as 72 registers hold (all of FC2's: 768 channels, 384 tiles 6.7 -> 7.2 us); the
// eight partial sums meet in LDS, and wave w < 4 finishes quad w of every lane's sixteen.  No stage, no barrier but one, and four times the
// workgroups of the ring kernel's smaller tiles, whose 430 clocks a stage of 128 bytes of K are their way through the L1 and LDS: see
// product_of_few_rows for the times.
template <int EPI, int SPW>
__global__ __launch_bounds__(512) void gemm_few_kernel(Geom G, GemmArgs A)
{
    touch_arguments<sizeof(Geom) + sizeof(GemmArgs)>();
    __shared__ v4i part[8][4][64];                                       // [wave][quad][lane]
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, j = lane & 31, g = lane >> 5;
    // the row tiles of a block of channels on one XCD, whose L2 then reads its weights once
    const int row_tiles = G.rows_total / 32, at = blockIdx.x >> 3, nb = (blockIdx.x & 7) + 8 * (at / row_tiles), tm = at % row_tiles;
    const int row = tm * 32 + j, branch = tm * 32 >= G.base_lo ? 1 : 0, N = A.N;
    constexpr int KS = 8 * SPW;
    const v4i *ap = (const v4i*)A.A + ((size_t)tm * KS + wave) * 64 + lane, *wp = A.Wp + ((size_t)nb * KS + wave) * 64 + lane;
    v4i av[SPW], wv[SPW];
#pragma unroll
    for (int s = 0; s < SPW; ++s) { av[s] = ap[s * 512]; wv[s] = wp[s * 512]; }
    const int n0 = nb * 32 + (wave & 3) * 8 + g * 4;                      // what the epilogue reads travels with them
    const float4 m = *(const float4*)(A.m[branch] + n0), bs = *(const float4*)(A.bias[branch] + n0);
    const int4 nc = *(const int4*)(A.negcorr[branch] + n0);
    const int canon = A.row_canon[row], pix = A.row_pix[row];
    float4 res = make_float4(0.f, 0.f, 0.f, 0.f);
    if (EPI == EPI_PROJ && pix >= 0) res = *(const float4*)(A.x + (size_t)pix * N + n0);
    if (EPI == EPI_FC2) res = *(const float4*)(A.resid + (size_t)row * N + n0);
    v16i acc = {};
#pragma unroll
    for (int s = 0; s < SPW; ++s) acc = mfma32(wv[s], av[s], acc);
#pragma unroll
    for (int qd = 0; qd < 4; ++qd) part[wave][qd][lane] = (v4i){acc[qd * 4], acc[qd * 4 + 1], acc[qd * 4 + 2], acc[qd * 4 + 3]};
    __syncthreads();
    if (wave >= 4) return;
    v4i sum = {nc.x, nc.y, nc.z, nc.w};                                  // -zp_in * colsum(W[n,:])
#pragma unroll
    for (int k = 0; k < 8; ++k) sum += part[k][wave][lane];
    if (A.tap_acc && canon >= 0) *(v4i*)(A.tap_acc + (size_t)canon * N + n0) = sum;
    const float f0 = fmaf((float)sum[0], m.x, bs.x), f1 = fmaf((float)sum[1], m.y, bs.y), f2 = fmaf((float)sum[2], m.z, bs.z), f3 = fmaf((float)sum[3], m.w, bs.w);
    const float4 o = make_float4(f0 + res.x, f1 + res.y, f2 + res.z, f3 + res.w);
    if (EPI == EPI_PROJ) *(float4*)(A.outf + (size_t)row * N + n0) = o;
    else if (pix >= 0) *(float4*)(A.y + (size_t)pix * N + n0) = o;
    if (A.tap_f && canon >= 0) *(float4*)(A.tap_f + (size_t)canon * N + n0) = o;
}

// ------------------------------------------------------------------ attention core
// For one (window, head) held by one wave.  S^T = K Q^T (A operand = key rows, B operand =
// query columns) leaves a lane with one query per query block and the keys in registers,
// so the softmax reduces in registers; the packed P codes are then directly the B operand
// of O^T = V^T P^T.  qf/kf: lane = token tb*32+j, 16 bytes = the lane half's 16 dims (any
// mapping, the same for q and k).  vt: lane = dim j, byte r of slab kb = V[kb*32 +
// mfma_row(r,g)][j], zero for keys >= 49.  Returns the zero-point corrected P.V sums (lane = query, register
// r = dim mfma_row(r,g)), zero-point corrected.  The wave runs NIB query blocks starting at block ib0 (both, or one of the
// two when a pair of waves shares the head).
// The P.V sums start at nzcsum[d] = -zp * sum of the V codes of dim d over the keys, formed once per dim by the caller
// (an integer multiply is a quarter-rate instruction; and starting the accumulators there costs no instruction, where
// subtracting afterwards took one per output element).
// (bias + mask) * log2e of a lane's query at its keys: quads kb * 8 + qd * 2 + g, and the last key (of the lower half only)
struct BiasRow {
    float4 quad[(TOK - 1) / 8];
    float last;
    // bq: query j of query block 0 at keys g*4 ..+3, in the [13 key quads][64 queries][4] table of the head and mask type
    __device__ __forceinline__ void request(const float4* bq, int g, int ib)
    {
#pragma unroll
        for (int k = 0; k < (TOK - 1) / 8; ++k) quad[k] = bq[k * 128 + ib * 32];
        last = bq[(TOK / 4 - g) * 64 + ib * 32].x;
    }
};
struct AttnCore {
    const float4* bq;         // see BiasRow::request
    float m2, c5;             // in vector registers, like qp's factor and addend
    QDev qp;
    const int* nzcsum;        // [HD], LDS
    bool floor;               // see exp2_pinned; scalar
    int32_t* tap_s;           // already offset to this (slot, head): [49][49]
    int8_t* tap_p;
};

// REQUEST: the bias is requested here (A.bq), otherwise the caller has done so
template <bool TAPS, bool REQUEST>
__device__ __forceinline__ v16i attention_core(const v4i& qf, const v4i (&kf)[2], const v4i (&vt)[2],
                                               const AttnCore& A, const BiasRow& bias, int j, int g, int ib)
{
    const v16i zero16 = {0};
    v16i o;
    {
        const int qi = ib * 32 + j;                               // this lane's query
        v16i s[2];                                                        // S^T tiles of this query block, per key block
        s[0] = mfma32(kf[0], qf, zero16);
        s[1] = mfma32(kf[1], qf, zero16);
        float lg[2][16];
        float mx = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 16; r += 4) {
                const int key = kb * 32 + (r >> 2) * 8;                   // + g*4
                float b[4] = {0.f, 0.f, 0.f, 0.f};
                if (key + 3 + 4 < TOK) {                                  // four keys, valid for both halves
                    const float4 b4 = REQUEST ? A.bq[(key / 4) * 64 + ib * 32] : bias.quad[key / 8];
                    b[0] = b4.x; b[1] = b4.y; b[2] = b4.z; b[3] = b4.w;
                } else if (key < TOK) b[0] = REQUEST ? A.bq[(key / 4 - g) * 64 + ib * 32].x : bias.last;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int kk = key + e + g * 4;
                    float v = -INFINITY;
                    if (key + e < TOK) {                                  // valid for at least one half
                        if (key + 7 < TOK || kk < TOK) v = fmaf((float)s[kb][r + e], A.m2, b[e]);
                        mx = fmaxf(mx, v);
                        if (TAPS && kk < TOK && qi < TOK && A.tap_s) A.tap_s[qi * TOK + kk] = s[kb][r + e];
                    }
                    lg[kb][r + e] = v;
                }
            }
        mx = half_max(mx);
        if (A.floor) {                                                    // masked pairs, infinities and NaN end here
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) lg[kb][r] = fmaxf(lg[kb][r] - mx, EXP2_FLOOR);
            mx = 0.0f;
        }
        double den = 0.0;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 16; r += 4) {
                const int key = kb * 32 + (r >> 2) * 8;
                if (key + 3 + 4 < TOK) {                                  // four keys, valid for both halves
                    float y[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[e] = lg[kb][r + e] - mx;
                    exp2_pinned<4>(y, A.c5);
                    den += sum4(y[0], y[1], y[2], y[3]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) lg[kb][r + e] = y[e];
                } else if (key < TOK) {                                   // the last key, of the lower half only
                    float y = lg[kb][r] - mx;
                    exp2_pinned<1>(&y, A.c5);
                    lg[kb][r] = key + g * 4 < TOK ? y : 0.0f;
                    den += (double)lg[kb][r];
                }
            }
        den = half_sum(den);
        const float rden = 1.0f / (float)den;
        v4i pk[2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            int wd[4];
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {
                int c[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int r = qd * 4 + e, key = kb * 32 + qd * 8 + e;
                    c[e] = 0;
                    if (key < TOK) {
                        const int kk = key + g * 4;
                        if (kk < TOK) {
                            c[e] = quant_code(lg[kb][r] * rden, A.qp);
                            if (TAPS && qi < TOK && A.tap_p) A.tap_p[qi * TOK + kk] = (int8_t)c[e];
                        }
                    }
                }
                wd[qd] = pack4(c[0], c[1], c[2], c[3]);
            }
            pk[kb] = (v4i){wd[0], wd[1], wd[2], wd[3]};
        }
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
            const int4 cz = *(const int4*)(A.nzcsum + qd * 8 + g * 4);
            o[qd * 4 + 0] = cz.x; o[qd * 4 + 1] = cz.y; o[qd * 4 + 2] = cz.z; o[qd * 4 + 3] = cz.w;
        }
        o = mfma32(vt[0], pk[0], o);
        o = mfma32(vt[1], pk[1], o);
    }
    return o;
}

// dequantization and requantization of the P.V sums; writes the codes of head `head` for the window's tokens to
// out[row0 + token][C] (and the taps)
template <bool TAPS, bool MAGIC>
__device__ __forceinline__ void attention_store(const v16i& o, const QDev& qo, float m_o,
                                                int j, int g, int ib, int head, int C, int8_t* out, int row0, int32_t* tap_o,
                                                int8_t* tap_code, size_t canon_row0, int pack = 0, int unsigned_pack = 0)
{
    {
        const int qi = ib * 32 + j;
        if (qi < TOK) {
            int code[4];
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {
                const int d0 = qd * 8 + g * 4;
                const int a0 = o[qd * 4 + 0], a1 = o[qd * 4 + 1], a2 = o[qd * 4 + 2], a3 = o[qd * 4 + 3];
                code[qd] = pack4(quant_code(sum_value<MAGIC>(a0) * m_o, qo), quant_code(sum_value<MAGIC>(a1) * m_o, qo),
                                 quant_code(sum_value<MAGIC>(a2) * m_o, qo), quant_code(sum_value<MAGIC>(a3) * m_o, qo));
                size_t ci = (canon_row0 + qi) * C + head * HD + d0;
                if (TAPS && tap_o) *(int4*)(tap_o + ci) = make_int4(sum_int<MAGIC>(a0), sum_int<MAGIC>(a1), sum_int<MAGIC>(a2), sum_int<MAGIC>(a3));
                if (TAPS && tap_code) *(int*)(tap_code + ci) = code[qd];
            }
            // The halves exchange, so that a lane stores its token's sixteen (packed: eight) consecutive bytes at once: four-byte
            // stores cost a write request each.
            if (pack == 0 || pack == PACK_FRAG) {
                if (unsigned_pack) {               // offset-binary in whole bytes, as a reader of packed codes expands them
                    const int flip = unsigned_pack == 1 ? 0x08080808 : 0x02020202, keep = unsigned_pack == 1 ? 0x0f0f0f0f : 0x03030303;
#pragma unroll
                    for (int qd = 0; qd < 4; ++qd) code[qd] = (code[qd] ^ flip) & keep;
                }
                const auto lo = __builtin_amdgcn_permlane32_swap(code[0], code[2], false, false);   // dims 0..3, 4..7 | 16..19, 20..23
                const auto hi = __builtin_amdgcn_permlane32_swap(code[1], code[3], false, false);   // 8..11, 12..15 | 24..27, 28..31
                const v4i all = {(int)lo[0], (int)lo[1], (int)hi[0], (int)hi[1]};
                const int ch = head * HD + g * 16;
                if (pack == 0) *(v4i*)(out + (size_t)(row0 + qi) * C + ch) = all;
                else *(v4i*)(out + frag_offset(row0 + qi, ch, C / 32)) = all;
            } else if (pack == 1) {                // out = first packed row of the region, row0 = row inside it
                int w[2];
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const int lo = (code[2 * p] ^ 0x08080808) & 0x0f0f0f0f, hi = (code[2 * p + 1] ^ 0x08080808) & 0x0f0f0f0f;
                    w[p] = lo | (hi << 4);
                }
                const auto both = __builtin_amdgcn_permlane32_swap(w[0], w[1], false, false);
                *(int2*)(out + (size_t)(row0 + qi) * (C / 2) + head * 16 + g * 8) = make_int2((int)both[0], (int)both[1]);
            } else if (pack == 2) {
                int w = 0;
#pragma unroll
                for (int qd = 0; qd < 4; ++qd) w |= ((code[qd] ^ 0x02020202) & 0x03030303) << (2 * qd);
                *(int*)(out + (size_t)(row0 + qi) * (C / 4) + head * 8 + g * 4) = w;
            }
        }
    }
}

// slot (high group of all images first, then the low group) -> branch, first row, canonical slot
__device__ __forceinline__ void slot_info(const Geom& G, int slot, int& branch, int& row0, int& canon_slot)
{
    const int n_hi = G.B * G.k_hi;
    if (slot < n_hi) { int b = G.by_hi(slot); branch = 0; row0 = slot * TOK; canon_slot = b * G.nW + (slot - b * G.k_hi); }
    else { int s = slot - n_hi, b = G.by_lo(s); branch = 1; row0 = G.base_lo + s * TOK; canon_slot = b * G.nW + G.k_hi + (s - b * G.k_lo); }
}

__device__ __forceinline__ int mask_type(const Geom& G, int w)
{
    if (G.shift == 0) return 0;
    int wr = G.by_nWc(w), wc = w - wr * G.nWc;
    return (wr == G.Hp / WS - 1 ? 2 : 0) + (wc == G.nWc - 1 ? 1 : 0);
}

// ------------------------------------------------------------------ K4 attention (unfused path)
// One wave per (window slot, head); q, k, v codes come from the row-major QKV buffer, V^T
// fragments from a transposing read of V staged in LDS.
__global__ __launch_bounds__(256) void attn_kernel(Geom G, AttnArgs A)
{
    __shared__ __attribute__((aligned(16))) int8_t vs[4][64 * HD];       // V tile per wave, [key][dim]
    __shared__ __attribute__((aligned(16))) int csum[4][HD];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, j = lane & 31, g = lane >> 5;
    const int item = blockIdx.x * 4 + wave;                              // slot * heads + head
    if (item >= G.n_slots * G.heads) return;
    const int slot = item / G.heads, head = item - slot * G.heads;
    int branch, row0, canon_slot;
    slot_info(G, slot, branch, row0, canon_slot);
    const int mtype = mask_type(G, A.perm[canon_slot]);
    const int C3 = 3 * G.C;
    const int8_t* base = A.qkv + (size_t)row0 * C3 + head * HD + g * 16;
    const v4i zero4 = {0, 0, 0, 0};
    v4i qf[2], kf[2];
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
        int t = tb * 32 + j;
        qf[tb] = t < TOK ? *(const v4i*)(base + (size_t)t * C3) : zero4;
        kf[tb] = t < TOK ? *(const v4i*)(base + (size_t)t * C3 + G.C) : zero4;
        v4i vv = t < TOK ? *(const v4i*)(base + (size_t)t * C3 + 2 * G.C) : zero4;
        *(v4i*)(&vs[wave][t * HD + g * 16]) = vv;
    }
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_wave_barrier();
    v4i vt[2];
    int cs = 0;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        int wd[4];
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
            int c[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) c[e] = vs[wave][(kb * 32 + qd * 8 + g * 4 + e) * HD + j];
            wd[qd] = pack4(c[0], c[1], c[2], c[3]);
            cs = __builtin_amdgcn_sdot4(wd[qd], 0x01010101, cs, false);
        }
        vt[kb] = (v4i){wd[0], wd[1], wd[2], wd[3]};
    }
    cs = half_sum(cs);
    if (g == 0) csum[wave][j] = -(A.qp[branch].zp * cs);
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_wave_barrier();
    AttnCore core;
    core.nzcsum = csum[wave];
    core.floor = (A.floor[branch] >> (mtype != 0)) & 1;
    core.c5 = in_vgpr(EXP2_C5);
    core.bq = A.bias2 + (size_t)(mtype * G.heads + head) * BIAS_QUADS * 64 + g * 64 + j;
    core.m2 = in_vgpr(A.m2[branch]);
    core.qp = in_vgpr(A.qp[branch]);
    const size_t tb = ((size_t)canon_slot * G.heads + head) * TOK * TOK;
    core.tap_s = A.tap_s ? A.tap_s + tb : nullptr;
    core.tap_p = A.tap_p ? A.tap_p + tb : nullptr;
#pragma unroll 1
    for (int ib = 0; ib < 2; ++ib) {
        const v16i o = attention_core<true, true>(ib ? qf[1] : qf[0], kf, vt, core, BiasRow(), j, g, ib);
        attention_store<true, false>(o, in_vgpr(A.qo[branch]), in_vgpr(A.m_o[branch]), j, g, ib, head, G.C, A.out, row0, A.tap_o, A.tap_code, (size_t)canon_slot * TOK, PACK_FRAG);
    }
}

// ------------------------------------------------------------------ LN1 of wide blocks
// Gather (shift folded in) + LN1 + quantize of the windows' tokens into MFMA operand fragments, per slot 64 token rows
// (49 and zeros), for the window kernel's CODES form; row bookkeeping, selection and pruned windows as there.  One
// workgroup per window and 256 / LPT tokens: few windows still make hundreds of workgroups.
template <int LPT, int NV, bool SCORED>
__global__ __launch_bounds__(256) void ln_window_kernel(Geom G, WinArgs A)
{
    touch_arguments<sizeof(Geom) + sizeof(WinArgs)>();
    constexpr int TP = 256 / LPT, C = LPT * NV * 4, KS = C / 32;
    __shared__ int red[4];
    const int tid = threadIdx.x, sub = tid % LPT, t = blockIdx.y * TP + tid / LPT, widx = blockIdx.x;
    int branch = 0, row0 = 0, canon_slot = 0, slot = widx, w, bimg;
    bool pruned = false;
    int pix = -1;
    float4 v[NV];
    auto gather = [&] {                                                   // needs the window only: ahead of its rank
        if (t < TOK) {
            const int wr = G.by_nWc(w), wc = w - wr * G.nWc, tr = t / WS, tc = t - tr * WS;
            int pr = wr * WS + tr + G.shift; if (pr >= G.Hp) pr -= G.Hp;
            int pc = wc * WS + tc + G.shift; if (pc >= G.Wp) pc -= G.Wp;
            pix = (pr < G.H && pc < G.W) ? (bimg * G.H + pr) * G.W + pc : -1;
        }
#pragma unroll
        for (int k = 0; k < NV; ++k) v[k] = pix >= 0 ? *(const float4*)(A.x + (size_t)pix * C + (k * LPT + sub) * 4) : make_float4(0.f, 0.f, 0.f, 0.f);
    };
    if (SCORED) {
        bimg = G.by_nW(widx);
        w = widx - bimg * G.nW;
        gather();
        const int rank = window_rank<256>(A.scores + (size_t)bimg * G.nW, G.nW, w, tid, red);
        if (tid == 0 && blockIdx.y == 0) A.perm_out[(size_t)bimg * G.nW + rank] = w;
        canon_slot = bimg * G.nW + rank;
        pruned = rank >= G.k_hi + G.k_lo;
        if (rank < G.k_hi) { slot = bimg * G.k_hi + rank; row0 = slot * TOK; }
        else { branch = 1; slot = bimg * G.k_lo + rank - G.k_hi; row0 = G.base_lo + slot * TOK; slot += G.B * G.k_hi; }
    } else if (widx < G.n_slots) {
        slot_info(G, widx, branch, row0, canon_slot);
        w = A.perm[canon_slot];
        bimg = G.by_nW(canon_slot);
    } else {
        const int kept = G.k_hi + G.k_lo, q = widx - G.n_slots;
        bimg = q / (G.nW - kept);
        w = A.perm[bimg * G.nW + kept + (q - bimg * (G.nW - kept))];
        pruned = true;
    }
    if (blockIdx.x == 0 && blockIdx.y == 0) {                             // the rows that pad each region to whole tiles belong to no window
        for (int r = G.rows_hi + tid; r < G.base_lo; r += 256) { A.row_pix[r] = -1; A.row_canon[r] = -1; }
        for (int r = G.base_lo + G.rows_lo + tid; r < G.rows_total; r += 256) { A.row_pix[r] = -1; A.row_canon[r] = -1; }
    }
    if (!SCORED) gather();
    Affine<NV> af;
    request_affine<LPT, NV>(af, A.params[branch], A.params[branch] + C, sub);
    if (pruned) {                                                         // Sec. 3.4: the features are forwarded
        if (pix >= 0) {
#pragma unroll
            for (int k = 0; k < NV; ++k) *(float4*)(A.y + (size_t)pix * C + (k * LPT + sub) * 4) = v[k];
        }
        return;
    }
    const int canon = canon_slot * TOK + t;
    if (sub == 0 && t < TOK) { A.row_pix[row0 + t] = pix; A.row_canon[row0 + t] = canon; }
    if (pix >= 0) token_layernorm<LPT, NV>(v, C, A.eps, af);              // padding enters as LN output 0
    const QDev q = in_vgpr(A.q_in[branch]);
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int ch = (k * LPT + sub) * 4;
        const int code = t < TOK ? pack4(quant_code(v[k].x, q), quant_code(v[k].y, q), quant_code(v[k].z, q), quant_code(v[k].w, q)) : 0;
        *(int*)(A.codes + frag_offset(slot * 64 + t, ch, KS)) = code;
        if (A.tap_a1 && t < TOK) *(int*)(A.tap_a1 + (size_t)canon * C + ch) = code;
    }
}

// ------------------------------------------------------------------ fused window kernel
// One workgroup per window slot (HG = 1) or per half of a window's heads (HG = 2: few windows, or more heads
// than a workgroup has waves; both halves repeat the gather + LN1 phase), one wave per head (QS = 1, NH waves)
// or a pair of waves per head (QS = 2: see win_roles; otherwise each wave projects one 32-token block to q, k and v; the pair exchanges
// through LDS what the other needs, and each runs the attention of its own query block: half the chain of dependent steps):
//   gather (shift folded into the index map) + LN1 + quantize, shared through LDS as MFMA
//   fragments -> per head: q, k (transposed product, lane = token) and v (plain product, lane =
//   dim) straight into operand registers -> attention core -> codes of the attention output.
// What bounds it on full CUs is the issue of instructions: a SIMD issues one vector instruction per four to five clocks for its
// even and one for its odd wave slots, and only one of the two at a time may be other than a simple one (see in_vgpr); a wave
// alone on its CU waits for the map, its weights and the bias.  Simple instructions in place of others in the softmax, no integer
// divisions, sixteen bytes a lane where the token slots behind the window are cleared, and sums over three, six or twelve lanes
// by quads: a pair of blocks on 4 x 256 x 256 x 128 458.6 -> 445.2 us, 2 x 50 x 84 x 384 (six blocks) 356.3 -> 347.4,
// 100 x 168 x 192 88.3 -> 86.5, one block on 56 x 56 x 96 19.7 -> 18.9.
template <int NH, int HG, int QS>
struct WinCfg {
    // lanes per token in the LN phase: one per wave (3 ... 16), so that the 49 tokens fit one pass
    // with about three quarters of the lanes busy; a wave holds 64/LPT whole groups
    static constexpr int LPT = NH * QS;
    static constexpr int GPW = 64 / LPT;                             // groups (tokens) per wave
    static constexpr int NV = NH * HG * 32 / (4 * LPT);              // float4 per lane = 8 * HG / QS
};
// Waves per SIMD the kernel is compiled for.  The loops over q / k and over the query blocks are real loops (unrolled, the
// scheduler spreads their loads over the whole kernel and wants 160 registers): with them a wave that owns a head needs 96
// to 118 registers instead of 160, one of a pair 74 to 78 where several workgroups share a CU.  A workgroup of six or twelve waves
// only gets a second place on a CU when its share per SIMD, rounded up, fits twice: 360 windows at C = 192 ran in two rounds of one
// workgroup per CU (24.6 us), now in one round (20.8 us); C = 256, 1444 windows: 83 -> 72 us.  (Three heads at five waves per SIMD
// spill none, six registers with scores; when they spilled two and four, and none at four waves, the pair of blocks on 1392 windows
// took 110.5 us at four waves and 108.0 at five.)
constexpr bool win_pairs_share(int NH, int HG) { return (NH == 6 && HG == 1) || NH * HG == 8; }   // pairs of waves, several workgroups on a CU
// Pairs that have the registers share the projections by roles: one wave takes q of all tokens, the other k, and v is split by
// tokens.  Each weight fragment of q and k then passes the L1 once and feeds two independent products, and its constants are read once.
// Against q, k and v each split by tokens, window kernel with LN1, us: 25 windows at C = 1024 20.0 -> 18.3, 24 at 768 15.7 -> 15.0, 4 at 512
// 12.4 -> 11.5, 96 at 384 15.2 -> 14.5, 196 at 192 14.8 -> 14.4, 64 at 128 7.8 -> 7.5; two blocks on 64 windows at C = 96 32.3 -> 31.9.
// Wide blocks, one wave per head (CODES, QS = 1): four waves per SIMD, at C = 768 three: a workgroup takes 42 of a CU's 128 LDS units of 1280 bytes.
// (With V's column sums in 512 bytes of their own it was 43, and a CU held two: two blocks on 90 windows 184.6 -> 178.6 us, 168 258 -> 254, 360
// 507 -> 496; 64 137.5 both.)  None spills, at 1024 with the weights four fragments ahead.  (Eight ahead spilled 33: 33 windows 25.5 -> 22.9 us, 48
// 29.6 -> 26.5, 100 48.6 -> 44.0, 200 85.6 -> 77.5, 288 109.5 -> 99.4.  At C = 512 and 768 four are equal up to 200 windows and 2 % behind beyond.)
// BESIDE (C = 96, beside a second chain; see window_beside): pairs without roles.  With their 126 registers a CU has places for two workgroups
// of six waves, both taken by the first chain, and what is left of the second one waits behind that chain's token kernel; with 87
// it has a third.  Four blocks on 722 windows 128 -> 124 us, 840 147 -> 134, 924 151 -> 139, 1012 164 -> 146.  And one wave per head at
// four waves per SIMD, where it spills none with scores either.
constexpr bool win_roles(int NH, int HG, int QS, bool CODES, bool BESIDE) { return QS == 2 && !BESIDE && (CODES || !win_pairs_share(NH, HG)); }
constexpr int win_waves_per_eu(int NH, int HG, int QS, bool CODES, bool BESIDE)
{
    if (CODES) return QS == 2 ? 2 : HG == 6 ? 3 : 4;
    if (QS == 2) return win_pairs_share(NH, HG) ? 6 : BESIDE ? 5 : NH == 6 ? 3 : 4;
    return NH * HG > 8 ? 3 : NH == 3 && !BESIDE ? 5 : 4;
}

// The window kernel's parameter block of one branch (see WinArgs::params), as a workgroup of NH heads holds it in LDS:
// LN1 gamma and beta (not with CODES), then the QKV epilogue constants of its own heads, per head [q|k|v][m|bias|-zp*colsum][32 dims]
template <int C, int NH, bool CODES> struct WinPrm {
    static constexpr int LN_G = 0, LN_B = C, HEADS = CODES ? 0 : 2 * C, PER_HEAD = 9 * HD, WORDS = HEADS + NH * PER_HEAD;
};

// CODES: the LN1 codes come ready from ln_window_kernel (wide blocks, whose heads are spread over many workgroups: each of
// them would repeat the whole gather and LayerNorm); the workgroup is given a slot and there are no pruned ones.
// WHOLE: the first half of block_kernel, whose workgroup goes on with the window's tokens: attention codes and pixels of the tokens stay
// in LDS (codes as operand fragments, a row block per 32 tokens), second_half() is called with the branch known, behind the write of this half's
// parameters to LDS.  False: the window is pruned and forwarded.
struct WholeLds {
    v4i *codes, *exchange;                                               // LN1's, then the attention's codes; what pairs of waves exchange
    int* pix;
};
template <int NH, bool TAPS, bool SCORED, int HG, int QS, bool CODES, bool MAGIC, bool BESIDE, bool WHOLE, typename Second>
__device__ __forceinline__ bool window_half(const Geom& G, const WinArgs& A, int& branch, const WholeLds& whole, Second second_half)
{
    constexpr int NHT = NH * HG;                                         // heads of the block; this workgroup runs NH of them
    constexpr int NW = NH * QS, NTB = 2 / QS;                            // waves; token blocks a wave projects to v and attends for
    constexpr bool ROLES = WHOLE || win_roles(NH, HG, QS, CODES, BESIDE);        // one wave of a pair projects all tokens to q, the other to k
    constexpr int NTQ = ROLES ? 2 : NTB, PAIR_SLOTS = ROLES ? 5 : 4;
    constexpr int C = NHT * 32, KS = NHT, LPT = WinCfg<NH, HG, QS>::LPT, NV = CODES ? 1 : WinCfg<NH, HG, QS>::NV, NT = NW * 64;
    constexpr int GPW = WinCfg<NH, HG, QS>::GPW;
    using PR = WinPrm<C, NH, CODES>;
    // the workgroups of a window on one XCD, whose L2 then reads the window once (1444 windows at C = 256: 339 -> 335 us the
    // pair); with CODES, one after another
    const int widx = HG == 1 ? blockIdx.x : CODES ? blockIdx.x / HG : blockIdx.x / (8 * HG) * 8 + blockIdx.x % 8;
    const int hg = HG == 1 ? 0 : CODES ? blockIdx.x % HG : blockIdx.x / 8 % HG;
    if (HG > 1 && !CODES && widx >= G.B * G.nW) return false;
    static_assert(CODES || NW * GPW >= TOK, "one pass must cover the window");
    __shared__ v4i own_a1s[WHOLE ? 1 : 2 * KS * 64];                     // LN1 codes as fragments [token block][k slab][lane]
    auto a1s = [&]() -> v4i* { if constexpr (WHOLE) return whole.codes; else return own_a1s; };
    __shared__ __attribute__((aligned(16))) float prm[PR::WORDS];        // this branch's LN1 affine and QKV epilogue constants
    constexpr bool SUMS_IN_PRM = CODES && QS == 1;                       // the V column sums of a wave's head take the place of its q multipliers, long read
    __shared__ __attribute__((aligned(16))) int csum[SUMS_IN_PRM ? 1 : NW][HD];
    __shared__ v4i own_kvx[QS == 2 && !WHOLE ? NH * PAIR_SLOTS * 64 : 1];   // k and v operands of a wave pair [head][k|v][token block][lane], with ROLES q of the second block
    auto kvx = [&]() -> v4i* { if constexpr (WHOLE) return whole.exchange; else return own_kvx; };
    __shared__ int csp[QS == 2 ? NH * 2 * HD : 1];                       // V column sums of each token block [head][block][dim]
    __shared__ int red[NW];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, j = lane & 31, g = lane >> 5;
    const int hw = QS == 1 ? wave : wave >> 1, tb0 = QS == 1 ? 0 : wave & 1;   // head inside the workgroup, first token block
    const int head = hg * NH + hw;
    // Weight fragments in flight.  STREAM: the fragments of q, k and v are one stream that starts under the LayerNorm phase and runs
    // on across the epilogues (each chain on its own starts with a wait for its first fragment: 100 x 168 x 192 87.0 -> 85.9 us,
    // 3 x 61 x 93 x 192 75.0 -> 73.3, backbone 621.8 -> 615).  Not where the registers are taken: three heads of a wave each spill
    // 17 to 26 of their 96, the pairs of C = 256 67 to 94 of their 80.  (Half a window's heads at C = 128 and 192 have 128, as few of
    // them share a CU: six blocks on 81 windows at C = 192 147 -> 133 us, three sets in turn of two blocks on 64 windows at
    // C = 128 36.7 -> 33.8.)
    constexpr bool STREAM = KS >= 12 || (HG == 1 ? !(NH == 3 && QS == 1) : KS < 8);
    constexpr int RING = !STREAM ? (KS < 6 ? KS : 6) : KS < 6 ? KS : KS == 6 ? (QS == 1 || WHOLE ? 6 : 3) : KS == 12 ? 6 : KS < 32 ? 8 : QS == 1 ? 4 : 16;
    static_assert(!STREAM || KS % RING == 0, "each chain starts at ring slot 0");
    constexpr int O_START = MAGIC ? SUM_MAGIC_BITS : 0;                  // of the P.V sums: 49 * 255 * 128 at most
    v4i ring[RING];
    const int role = ROLES ? __builtin_amdgcn_readfirstlane(tb0) : 0;
    auto weights_of = [&](int which) { return A.Wqkv + (size_t)(which * NHT + head) * KS * 64 + lane; };
    // SCORED: the workgroup is given a window and finds its own place in the selection (its rank
    // under the total order of the scores); otherwise it is given a slot and looks the window up.
    int row0 = 0, canon_slot = 0, w, bimg = 0;
    branch = 0;
    if (STREAM && CODES) {
        const v4i* wp = weights_of(role);
#pragma unroll
        for (int d = 0; d < RING; ++d) ring[d] = wp[d * 64];
    }
    if (SCORED) {
        bimg = G.by_nW(widx);
        w = widx - bimg * G.nW;
    } else if (widx < G.n_slots) {
        slot_info(G, widx, branch, row0, canon_slot);
        w = A.perm[canon_slot];
        bimg = G.by_nW(canon_slot);
    } else {                              // workgroups past the computed slots: pruned windows (Sec. 3.4), features forwarded
        if (hg != 0) return false;
        const int kept = G.k_hi + G.k_lo, q = widx - G.n_slots, b = q / (G.nW - kept);
        const int wp = A.perm[b * G.nW + kept + (q - b * (G.nW - kept))];
        const int wr = G.by_nWc(wp), wc = wp - wr * G.nWc;
        for (int i = tid; i < TOK * (C / 4); i += NT) {
            const int tt = i / (C / 4), k = i - tt * (C / 4), tr = tt / WS, tc = tt - tr * WS;
            int pr = wr * WS + tr + G.shift; if (pr >= G.Hp) pr -= G.Hp;
            int pc = wc * WS + tc + G.shift; if (pc >= G.Wp) pc -= G.Wp;
            if (pr < G.H && pc < G.W) {
                const size_t off = ((size_t)(b * G.H + pr) * G.W + pc) * C + k * 4;
                *(float4*)(A.y + off) = *(const float4*)(A.x + off);
            }
        }
        return false;
    }
    // The rows that pad each region to whole tiles belong to no window: the first workgroup marks them
    // (pixel -1, slot-major row -1) for the kernels of the seven-kernel path, which read the marks of every row.
    if (!CODES && !WHOLE && blockIdx.x == 0) {
        for (int r = G.rows_hi + tid; r < G.base_lo; r += NT) { A.row_pix[r] = -1; A.row_canon[r] = -1; }
        for (int r = G.base_lo + G.rows_lo + tid; r < G.rows_total; r += NT) { A.row_pix[r] = -1; A.row_canon[r] = -1; }
    }
    int* a1w = (int*)a1s();
    // dword index of (token slot s, channel c with c%4==0) in the fragment layout (k = channel, natural order)
    auto frag_dw = [&](int s, int c) { return ((((s >> 5) * KS + (c >> 5)) * 64 + ((c & 31) >> 4) * 32 + (s & 31)) << 2) + ((c & 15) >> 2); };
    static_assert(CODES || NT >= 32 * KS, "one pass must clear the token slots behind the window");
    if (!CODES && tid < 32 * KS && (tid & 15) < 64 - TOK)                 // the fifteen of every half slab, sixteen bytes a lane
        a1s()[(KS + (tid >> 5)) * 64 + ((tid >> 4) & 1) * 32 + TOK - 32 + (tid & 15)] = (v4i){0, 0, 0, 0};
    const int grp = lane / LPT, sub = lane - grp * LPT, first = lane - sub;
    const int t = !CODES && grp < GPW ? wave * GPW + grp : TOK;          // lanes beyond the last whole group idle
    int pix = -1;
    float4 v[NV];
    if (t < TOK) {                                                       // gather: the loads need the window only
        const int wr = G.by_nWc(w), wc = w - wr * G.nWc, tr = t / WS, tc = t - tr * WS;
        int pr = wr * WS + tr + G.shift; if (pr >= G.Hp) pr -= G.Hp;
        int pc = wc * WS + tc + G.shift; if (pc >= G.Wp) pc -= G.Wp;
        pix = (pr < G.H && pc < G.W) ? (bimg * G.H + pr) * G.W + pc : -1;
        if (pix >= 0) {
            const float* src = A.x + (size_t)pix * C;
#pragma unroll
            for (int k = 0; k < NV; ++k) v[k] = *(const float4*)(src + (k * LPT + sub) * 4);
        }
    }
    if (SCORED) {
        const int rank = window_rank<NT>(A.scores + (size_t)bimg * G.nW, G.nW, w, tid, red);
        if (tid == 0 && hg == 0) A.perm_out[(size_t)bimg * G.nW + rank] = w;
        if (rank >= G.k_hi + G.k_lo) {                                    // pruned (Sec. 3.4): forward the features
            if (pix >= 0 && hg == 0) {
                float* dst = A.y + (size_t)pix * C;
#pragma unroll
                for (int k = 0; k < NV; ++k) *(float4*)(dst + (k * LPT + sub) * 4) = v[k];
            }
            return false;                                                 // the whole workgroup
        }
        canon_slot = bimg * G.nW + rank;
        if (rank < G.k_hi) { branch = 0; row0 = (bimg * G.k_hi + rank) * TOK; }
        else { branch = 1; row0 = G.base_lo + (bimg * G.k_lo + rank - G.k_hi) * TOK; }
    }
    {   // the branch is known: its parameter block goes to LDS (requested now, so that it travels with the map)
        const float4* src = (const float4*)A.params[branch];
        constexpr int PV = PR::WORDS / 4, PVT = (PV + NT - 1) / NT;
        float4 pv[PVT];
#pragma unroll
        for (int k = 0; k < PVT; ++k) {
            const int i = min(tid + k * NT, PV - 1);
            pv[k] = src[HG > 1 && i >= PR::HEADS / 4 ? i + hg * (NH * PR::PER_HEAD / 4) + (CODES ? 2 * C / 4 : 0) : i];
        }
        if (CODES) {                                                      // operand fragments straight to LDS
            const int wv = __builtin_amdgcn_readfirstlane(wave);
            for (int f = wv; f < 2 * KS; f += NW)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(A.codes + ((size_t)widx * 2 * KS + f) * 1024 + lane * 16),
                                                 (__attribute__((address_space(3))) void*)(a1s() + f * 64), 16, 0, 0);
        }
        if (STREAM && !CODES) {
            const v4i* wp = weights_of(role);
#pragma unroll
            for (int d = 0; d < RING; ++d) ring[d] = wp[d * 64];
        }
#pragma unroll
        for (int k = 0; k < PVT; ++k) if (tid + k * NT < PV) ((float4*)prm)[tid + k * NT] = pv[k];
        second_half();
    }
    if (CODES) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // the direct loads have landed
    __syncthreads();                                                     // parameter block visible
    if (t < TOK) {
        const int canon = canon_slot * TOK + t;
        if (WHOLE) { if (sub == 0) whole.pix[t] = pix; }
        else if (sub == 0 && hg == 0) { A.row_pix[row0 + t] = pix; A.row_canon[row0 + t] = canon; }
        if (pix >= 0) {
            token_layernorm<LPT, NV>(v, C, A.eps, prm + PR::LN_G, prm + PR::LN_B, sub, first);
        } else {
#pragma unroll
            for (int k = 0; k < NV; ++k) v[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        const QDev q = in_vgpr(A.q_in[branch]);
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            if (NV > 8 && k % 4 == 0) __builtin_amdgcn_sched_barrier(0);
            const int ch = (k * LPT + sub) * 4;
            int code = pack4(quant_code(v[k].x, q), quant_code(v[k].y, q), quant_code(v[k].z, q), quant_code(v[k].w, q));
            // four vectors on, the fragment address is a constant further (32 channels are 1 KB of fragments, and a token's slabs
            // follow one another in whole vectors of sixteen channels): at most four addresses are formed
            a1w[frag_dw(t, ((k & 3) * LPT + sub) * 4) + (k >> 2) * LPT * 128] = code;
            if (TAPS && A.tap_a1 && hg == 0) *(int*)(A.tap_a1 + (size_t)canon * C + ch) = code;
        }
    }
    if (!CODES) __syncthreads();
    // The B operand (LN1 fragments) is read from LDS inside the chain and the weight fragments come through a short ring of
    // loads: held in registers instead (24 to 64 of them) they cost the kernel its fourth and fifth wave per SIMD.
    // acc[tb] += (weights as A operand ? W * act^T : act * W^T) over the whole K; next: where the stream goes on
    auto chain = [&](auto BLOCKS, const v4i* wp, const v4i* next, v16i* acc, bool weights_first) {   // both token blocks, or the wave's own
        constexpr int PF = STREAM ? 3 : 1, NTB = decltype(BLOCKS)::value; // LDS reads ahead (the scheduler's own business otherwise)
        v4i xv[PF][NTB];
        auto operand = [&](int ks) {
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb) xv[ks % PF][tb] = a1s()[(((ROLES && NTB == 2 ? 0 : tb0) + tb) * KS + ks) * 64 + lane];
        };
        if (STREAM) {
#pragma unroll
            for (int d = 0; d < PF; ++d) operand(d);
        } else {
#pragma unroll
            for (int d = 0; d < RING; ++d) ring[d] = wp[d * 64];
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (!STREAM) operand(ks);
            const v4i wv = ring[ks % RING];
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb) acc[tb] = weights_first ? mfma32(wv, xv[ks % PF][tb], acc[tb]) : mfma32(xv[ks % PF][tb], wv, acc[tb]);
            if (ks + RING < KS) ring[ks % RING] = wp[(ks + RING) * 64];
            else if (STREAM && next) ring[ks % RING] = next[(ks + RING - KS) * 64];
            if (STREAM) {                                                 // product, request into the slot just used, LDS read: see gemm_tile_kernel
                if (ks + PF < KS) operand(ks + PF);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    const size_t canon_row0 = (size_t)canon_slot * TOK;
    auto column_sums = [&]() -> int* { return SUMS_IN_PRM ? (int*)(prm + PR::HEADS + hw * PR::PER_HEAD) : csum[wave]; };
    v4i qk[2][NTQ] = {};                                                 // [q|k][token block]; with ROLES the wave's own in [1]
#pragma unroll 1
    for (int which = role; which < (ROLES ? role + 1 : 2); ++which) {
        asm volatile("" ::: "memory");                                    // the B operand is read from LDS each time: keep the reads in the loop
        const int nb = which * NHT + head;
        const float* pm = prm + PR::HEADS + hw * PR::PER_HEAD + which * (3 * HD);
        const QDev qq = in_vgpr(A.q_qkv[branch][which]);
        const v4i* wp = weights_of(which);
        auto start = [&](v16i& acc) {                                     // accumulators start at -zp * colsum
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {
                const int4 t4 = *(const int4*)((const int*)pm + 2 * HD + qd * 8 + g * 4);
                acc[qd * 4 + 0] = t4.x; acc[qd * 4 + 1] = t4.y; acc[qd * 4 + 2] = t4.z; acc[qd * 4 + 3] = t4.w;
            }
        };
        auto finish = [&](int tb, const v16i& acc) {                      // dequantize, requantize, keep as operand
            int wd[4];
            const int tok = ((NTQ == 2 ? 0 : tb0) + tb) * 32 + j;
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {
                const int n0 = nb * 32 + qd * 8 + g * 4;
                const float4 m = *(const float4*)(pm + qd * 8 + g * 4), bs = *(const float4*)(pm + HD + qd * 8 + g * 4);
                const int a0 = acc[qd * 4 + 0], a1 = acc[qd * 4 + 1], a2 = acc[qd * 4 + 2], a3 = acc[qd * 4 + 3];
                wd[qd] = pack4(quant_code(fmaf(sum_value<MAGIC>(a0), m.x, bs.x), qq), quant_code(fmaf(sum_value<MAGIC>(a1), m.y, bs.y), qq),
                               quant_code(fmaf(sum_value<MAGIC>(a2), m.z, bs.z), qq), quant_code(fmaf(sum_value<MAGIC>(a3), m.w, bs.w), qq));
                if (TAPS && tok < TOK) {
                    if (A.tap_acc) *(int4*)(A.tap_acc + (canon_row0 + tok) * (3 * C) + n0) = make_int4(sum_int<MAGIC>(a0), sum_int<MAGIC>(a1), sum_int<MAGIC>(a2), sum_int<MAGIC>(a3));
                    if (A.tap_qkv) *(int*)(A.tap_qkv + (canon_row0 + tok) * (3 * C) + n0) = wd[qd];
                }
            }
            if (!ROLES) qk[0][tb] = qk[1][tb];                            // the second trip moves q to its place (a select costs twice a move)
            qk[1][tb] = (v4i){wd[0], wd[1], wd[2], wd[3]};
        };
        v16i acc[NTQ];
        start(acc[0]);
        if (NTQ == 2) acc[NTQ - 1] = acc[0];
        chain(std::integral_constant<int, NTQ>(), wp, weights_of(ROLES ? 2 : which + 1), acc, true);
#pragma unroll
        for (int tb = 0; tb < NTQ; ++tb) finish(tb, acc[tb]);
    }
    // a pair of waves requests its bias ahead of the exchange, where the registers are free
    constexpr bool BIAS_EARLY = QS == 2 && (WHOLE || CODES || !win_pairs_share(NH, HG));
    BiasRow bias;
    v4i vt[2];
    {
        const int nb = 2 * NHT + head, n = nb * 32 + j;                   // this lane's output channel (dim j of the head)
        const v4i* wp = weights_of(2);
        const float* pm = prm + PR::HEADS + hw * PR::PER_HEAD + 2 * (3 * HD) + j;
        const float m = pm[0], bs = pm[HD];
        const int nc = __float_as_int(pm[2 * HD]);
        const QDev qv = in_vgpr(A.q_qkv[branch][2]);
        int cs = 0;
        auto finish = [&](int tb, const v16i& acc) {
            int wd[4];
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {
                int c[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int tok = (tb0 + tb) * 32 + qd * 8 + g * 4 + e;
                    c[e] = 0;
                    if (QS == 2 || tb * 32 + qd * 8 + e < TOK) {      // known at compile time when the wave runs both blocks
                        if (tok < TOK) {
                            c[e] = quant_code(fmaf(sum_value<MAGIC>(acc[qd * 4 + e]), m, bs), qv);
                            if (TAPS && A.tap_acc) A.tap_acc[(canon_row0 + tok) * (3 * C) + n] = sum_int<MAGIC>(acc[qd * 4 + e]);
                            if (TAPS && A.tap_qkv) A.tap_qkv[(canon_row0 + tok) * (3 * C) + n] = (int8_t)c[e];
                        }
                    }
                }
                wd[qd] = pack4(c[0], c[1], c[2], c[3]);
                cs = __builtin_amdgcn_sdot4(wd[qd], 0x01010101, cs, false);
            }
            vt[tb] = (v4i){wd[0], wd[1], wd[2], wd[3]};
        };
        v16i acc[NTB];
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][r] = nc;
        if (NTB == 2) acc[NTB - 1] = acc[0];
        chain(std::integral_constant<int, NTB>(), wp, nullptr, acc, false);
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) finish(tb, acc[tb]);
        if (BIAS_EARLY)                                                   // under the exchange
            bias.request(A.bias2 + (size_t)(mask_type(G, w) * NHT + head) * BIAS_QUADS * 64 + g * 64 + j, g, tb0);
        cs = half_sum(cs);
        if (QS == 1) {
            if (g == 0) column_sums()[j] = O_START - A.qp[branch].zp * cs;
        } else {                                                          // the pair exchanges its halves of K, V and the sums
            if (!ROLES) kvx()[((hw * 2 + 0) * 2 + tb0) * 64 + lane] = qk[1][0];
            else if (role) { kvx()[(hw * PAIR_SLOTS + 0) * 64 + lane] = qk[1][0]; kvx()[(hw * PAIR_SLOTS + 1) * 64 + lane] = qk[1][NTQ - 1]; }
            else kvx()[(hw * PAIR_SLOTS + PAIR_SLOTS - 1) * 64 + lane] = qk[1][NTQ - 1];
            kvx()[(hw * PAIR_SLOTS + 2 + tb0) * 64 + lane] = vt[0];
            if (g == 0) csp[(hw * 2 + tb0) * HD + j] = cs;
            __syncthreads();
            if (g == 0) column_sums()[j] = O_START - A.qp[branch].zp * (csp[(hw * 2) * HD + j] + csp[(hw * 2 + 1) * HD + j]);
        }
    }
    v4i kf[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        kf[kb] = QS == 1 ? qk[1][kb % NTQ] : kvx()[(hw * PAIR_SLOTS + kb) * 64 + lane];
        if (QS == 2) vt[kb] = kvx()[(hw * PAIR_SLOTS + 2 + kb) * 64 + lane];
    }
    if (ROLES) qk[0][0] = role ? kvx()[(hw * PAIR_SLOTS + PAIR_SLOTS - 1) * 64 + lane] : qk[1][0];
    __builtin_amdgcn_s_waitcnt(0xc07f);                                   // lgkmcnt(0): the wave's own column sums are in LDS
    __builtin_amdgcn_wave_barrier();
    const int mtype = mask_type(G, w);
    AttnCore core;
    core.floor = (A.floor[branch] >> (mtype != 0)) & 1;
    core.c5 = in_vgpr(EXP2_C5);
    core.nzcsum = column_sums();
    core.bq = A.bias2 + (size_t)(mtype * NHT + head) * BIAS_QUADS * 64 + g * 64 + j;
    core.m2 = in_vgpr(A.m2[branch]);
    core.qp = in_vgpr(A.qp[branch]);
    const size_t tbase = ((size_t)canon_slot * NHT + head) * TOK * TOK;
    core.tap_s = A.tap_s ? A.tap_s + tbase : nullptr;
    core.tap_p = A.tap_p ? A.tap_p + tbase : nullptr;
    // the low region's rows may be packed (dense, after the high region); operand fragments are the same for both branches
    const int pack = WHOLE ? PACK_FRAG : A.out_pack == PACK_FRAG || branch ? A.out_pack : 0;
    const bool dense = pack == 1 || pack == 2;
    int8_t* out = WHOLE ? (int8_t*)whole.codes : A.out + (dense ? (size_t)G.base_lo * C : 0);
    const int orow0 = WHOLE ? 0 : row0 - (dense ? G.base_lo : 0);
#pragma unroll 1
    for (int ib = tb0; ib < tb0 + NTB; ++ib) {
        asm volatile("" ::: "memory");
        const v16i o = attention_core<TAPS, !BIAS_EARLY>(NTB == 2 && ib ? qk[0][NTB - 1] : qk[0][0], kf, vt, core, bias, j, g, ib);
        attention_store<TAPS, MAGIC>(o, in_vgpr(A.qo[branch]), in_vgpr(A.m_o[branch]), j, g, ib, head, C, out, orow0, A.tap_o, A.tap_code, canon_row0, pack, WHOLE && branch ? A.out_pack : 0);
    }
    return true;
}

template <int NH, bool TAPS, bool SCORED, int HG, int QS, bool CODES, bool MAGIC, bool BESIDE>
__global__ __launch_bounds__(NH * QS * 64) __attribute__((amdgpu_waves_per_eu(win_waves_per_eu(NH, HG, QS, CODES, BESIDE)))) void window_kernel(Geom G, WinArgs A)
{
    if (CODES || HG == 2 || (QS == 2 && NH <= 4)) touch_arguments<sizeof(Geom) + sizeof(WinArgs)>();   // few workgroups
    int branch;
    window_half<NH, TAPS, SCORED, HG, QS, CODES, MAGIC, BESIDE, false>(G, A, branch, WholeLds(), [] {});
}

// ------------------------------------------------------------------ fused token kernel
// One workgroup per tile of 32*RB gathered rows (RB 32-row blocks share every weight fragment), one wave per 32-channel
// block (NH = C/32 = 3, 4, 6, 8 or 12 waves):
//   proj + first residual (wave w owns channels 32w..32w+31) -> LN2 with statistics exchanged through LDS -> quantize -> FC1 +
//   GELU + quantize, codes to LDS as fragments -> FC2 + second residual -> scatter to the map.
// The weight fragments of the whole kernel form ONE stream per wave that is requested RING fragments ahead across every phase
// boundary; the per-branch parameter block and the GELU table (of steps, or with SHORT off of cubics) sit in LDS.  The FFN runs in
// four chunks of NH hidden blocks: FC1 + GELU + quantize of a chunk goes to one of two LDS buffers, then FC2 accumulates that chunk.
// With two row blocks h is parked in the output map between the first and the second residual (the same thread writes and re-reads the
// same address).
// Bound: vector instructions (57 to 62 % of the cycles) and LDS reads (48 to 54 %) that do not overlap fully at C = 96 and 128 on large
// maps, the weights at 64 bytes per clock and CU at C = 384, the chain of phases on few tiles.  Against a form with the chunks unrolled
// and FC1's weights a block ahead, which the three, four and eight waves had: stage of two blocks on 8 x 1392 windows at C = 96, 5476
// at C = 128 and 1444 at C = 256 3 % shorter, 64 windows at C = 256 58.9 -> 52.7 us.
// SHORT: the table of steps and the sums of the projection and FC1 without a conversion, together, or neither: a block whose FC2 input has
// no table (8 bits on a range narrower than about 0.5) in one branch, or whose sums are not bounded, runs as it did before both.
// LN2's partial sums are read together and each by one half of the lanes, for both row blocks before either goes on, and the
// parked h is requested ahead of the last products: 2 x 50 x 84 x 384 (six blocks) 347.4 -> 340.6 us, of 64-row tiles' 72 k clocks
// these phases had taken 15 k and 7 k.
// Waves per SIMD it is compiled for: 128 registers take it without spills up to six waves (106 to 124 wanted), at eight waves
// with six spilled; at five waves per SIMD the spills at C = 96 cost more than the fifth wave gives; twelve need 160 and have a
// CU to themselves.
constexpr int tok_waves_per_eu(int NH) { return NH == 12 ? 3 : 4; }
// word offsets inside the parameter block of one branch (see TokArgs::params)
template <int C> struct TokPrm {
    static constexpr int F = 4 * C;
    static constexpr int P_M = 0, P_B = C, P_NC = 2 * C, LN_G = 3 * C, LN_B = 4 * C, F2_M = 5 * C, F2_B = 6 * C,
                         F2_NC = 7 * C, F1_M = 8 * C, F1_B = 8 * C + F, F1_NC = 8 * C + 2 * F, WORDS = (8 * C + 3 * F + 255) / 256 * 256;   // whole 1 KB pieces
};

// 64 lanes x 16 bytes from memory straight into LDS (src per lane, dst the wave's 1 KB)
__device__ __forceinline__ void to_lds(const void* src, void* dst)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}
// requests the branch's parameter block and the GELU table (1 KB pieces) of a token kernel of NH waves
template <int NH, int WORDS>
__device__ __forceinline__ void token_stage(const float* params, const float4* gelu, int gelu_pieces, float* prm, float4* gtab, int wave, int lane)
{
    constexpr int PIECES = WORDS / 256;
#pragma unroll
    for (int p0 = 0; p0 < PIECES; p0 += NH)
        if (p0 + NH <= PIECES || p0 + wave < PIECES) to_lds(params + (p0 + wave) * 256 + lane * 4, prm + (p0 + wave) * 256);
    for (int p = NH - 1 - wave; p < gelu_pieces; p += NH) to_lds(gelu + p * 64 + lane, gtab + p * 64);   // the last waves have the fewest of the others
}

// LN2's partial sums, up to eight waves in the room of the hidden codes: the last sum is read ahead of the barrier in front of the FFN.
// LDS is given out in one piece of whole units, 128 of 1280 bytes, so a workgroup's size decides which ones share a CU.  At C = 96 five take
// 5 x 24 (with sums of their own 5 x 26, and a CU held four: 200 x 336 98.5 -> 95.4 us, 8 x 200 x 336 606 -> 594).  At C = 256 a second
// token workgroup has to fit behind one that lies behind a window workgroup of the other chain, 33 + 2 x 46.  (With the sums in 4 KB of
// their own the table of steps made it 49, and such a CU had one token workgroup until both were through: six blocks, two chains, 200
// windows 219.7 -> 203.3 us, 288 240 -> 229, 480 343 -> 321, 612 402 -> 401; before the table, 40 units, 211, 240, 332, 413.)  Twelve
// waves have a CU to themselves, and with 64 rows the shared room costs 12 spilled registers: two blocks on 840 windows 330 -> 358 us.
constexpr bool tok_sums_in_codes(int NH) { return NH <= 8; }
// LDS of a workgroup whose waves take GROUPS tiles of 32 * RB rows side by side, NH waves each.  In this order, table first, C = 384 is
// 0.4 % shorter than with the codes first (300 windows, two blocks 149.5 -> 148.8 us), other widths equal.
template <int NH, int RB, int GROUPS, bool SHORT>
struct TokLds {
    float4 gtab[SHORT ? GELU_STEP_PIECES * 64 : GELU_TAB];
    __attribute__((aligned(16))) float prm[TokPrm<NH * 32>::WORDS];
    v4i gs[GROUPS == 1 ? 1 : 0][2][NH * RB * 64];                      // [buffer][hidden block of the chunk][row block][lane]
    v4i actf[GROUPS][RB * NH * 64];                                    // [row block][k slab][lane]
};

// WHOLE: the second half of block_kernel: tile `group` of the window that the workgroup has in LDS, whose parameters and table are requested.
template <int NH, int RB, bool TAPS, bool SHORT, int GROUPS, bool WHOLE>
__device__ __forceinline__ void token_half(const Geom& G, const TokArgs& A, TokLds<NH, RB, GROUPS, SHORT>& S, int branch, const int* whole_pix, v4i (*whole_gs)[2][NH * RB * 64])
{
    constexpr int C = NH * 32, KS = NH, HB = 4 * NH, F = 4 * C;
    constexpr int RING = NH < 8 ? NH : NH == 12 && RB == 1 ? 12 : 8;               // fragments in flight per wave
    constexpr bool PARK_H = RB >= 2 && !TAPS;                         // taps need h of padded tokens too, which have no pixel
    static_assert((2 * KS) % RING == 0 && RING <= KS, "phases 2k start at ring slot 0, phases 2k+1 at slot KS % RING");
    constexpr int SLOT_ODD = KS % RING;
    using PR = TokPrm<C>;
    const int lane = threadIdx.x & 63, all_waves = threadIdx.x >> 6, group = GROUPS == 1 ? 0 : __builtin_amdgcn_readfirstlane(all_waves / NH);
    const int wave = GROUPS == 1 ? all_waves : all_waves - group * NH, j = lane & 31, g = lane >> 5;
    v4i* const actf = S.actf[group];
    auto& gs = WHOLE ? whole_gs[group] : S.gs[0];
    __shared__ double own_sums[tok_sums_in_codes(NH) ? 1 : 2 * NH * 32 * RB];
    auto& part = *reinterpret_cast<double (*)[2][NH][32 * RB]>(tok_sums_in_codes(NH) ? (double*)gs[0] : own_sums);
    static_assert(GROUPS == 1 || tok_sums_in_codes(NH), "sums of a group's own");
    static_assert(!tok_sums_in_codes(NH) || sizeof(part) <= sizeof(gs[0]), "in one buffer of the hidden codes");
    float* const prm = S.prm;
    float4* const gtab = S.gtab;
    const int row_base = WHOLE ? 0 : blockIdx.x * (32 * RB);
    if (!WHOLE) branch = row_base >= G.base_lo ? 1 : 0;               // a tile never straddles the regions: scalar
    const int nb = wave;
    const int* prmi = (const int*)prm;
    // The wave's weight stream, phase by phase (every phase has KS = NH fragments): projection block, FC1 block of
    // chunk 0, then per chunk c = 1..3 the FC1 block of chunk c followed by the FC2 fragments of chunk c-1, and the
    // FC2 fragments of chunk 3 at the end.  FC2 of a chunk is issued one chunk late, with the GELU arithmetic of the next chunk
    // between its steps: the weights then arrive (64 bytes per clock and CU bound this kernel at C = 384) while it runs
    // (C = 384, 32-row tiles 24.0 -> 23.4 us, 64-row tiles 39.5 -> 38.6; C = 192 26.1 -> 25.5).
    const v4i* wproj = A.Wproj + (size_t)nb * KS * 64 + lane;
    auto w1_of = [&](int chunk) { return A.W1 + ((size_t)(chunk * NH + wave) * KS) * 64 + lane; };
    auto w2_of = [&](int chunk) { return A.W2 + ((size_t)nb * HB + chunk * NH) * 64 + lane; };
    // Staging: the attention codes of the tile as operand fragments, the parameter block and the GELU table.  What is a plain
    // copy goes straight to LDS and everything is requested before anything is waited for (piece by piece, load and LDS
    // write in a loop, the staging was a chain of round trips: 3.3 us of a tile's 14 at C = 192).
    const int swave = __builtin_amdgcn_readfirstlane(wave);
    const int pack = branch && !WHOLE ? A.ao_pack : 0;                 // packed low-branch codes: scalar per tile
    int2 pc[RB];
    if (!pack && !WHOLE) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)                                // fragment (rb, slab = wave), lane (half g, row j)
            to_lds(A.ao + (size_t)(row_base + rb * 32 + j) * C + swave * 32 + g * 16, actf + (rb * KS + swave) * 64);
    }
    if (pack) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
            pc[rb] = packed_codes(A.ao + (size_t)G.base_lo * C + (size_t)(row_base - G.base_lo + rb * 32 + j) * (C >> pack), pack, wave, g);
    }
    int pix[RB];
    bool valid[RB];
    size_t canon[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int row = row_base + rb * 32 + j;
        if (WHOLE) { valid[rb] = group * 32 + j < TOK; continue; }     // (the pixel is in LDS behind the barrier)
        valid[rb] = branch ? (row - G.base_lo < G.rows_lo) : (row < G.rows_hi);
        pix[rb] = A.row_pix[row];
        canon[rb] = (TAPS && valid[rb]) ? (size_t)A.row_canon[row] : 0;
    }
    if (!WHOLE) token_stage<NH, PR::WORDS>(A.params[branch], SHORT ? (const float4*)A.steps[branch] : A.gelu_tab, SHORT ? A.step_pieces[branch] : GELU_TAB / 64, prm, gtab, swave, lane);
    asm volatile("" ::: "memory");                                     // the weight stream is requested behind them
    v4i ring[RING];
#pragma unroll
    for (int d = 0; d < RING; ++d) ring[d] = wproj[d * 64];
    asm volatile("" ::: "memory");
    // acc[rb] += W * operand^T over one phase.  Weights come from the ring (SLOT0 = ring slot of the phase's first
    // fragment); after fragment i is used, the fragment RING places further down the stream is requested into its slot: from
    // this phase (cur) or from the start of the next one (nxt; LAST: the end of the stream).  Operand fragment i of row
    // block rb: b[(rb*rb_stride + i*i_stride)*64 + lane], read PF steps ahead.  The steps keep their order (product, request,
    // LDS read): see gemm_tile_kernel.
    // A phase starts on operands that the phase before it requested (FC2's behind the last step of FC1, FC1's ahead of the barrier: LN2's
    // codes no longer change): 100 x 168 x 192 86.6 -> 86.2 us, backbone 621 -> 619.
    constexpr int PF = 2;
    v4i bq[PF][RB];
    auto request = [&](const v4i* b, int rb_stride, int i_stride) {
#pragma unroll
        for (int i = 0; i < PF; ++i)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) bq[i][rb] = b[(rb * rb_stride + i * i_stride) * 64 + lane];
    };
    auto run = [&](auto SLOT0, auto LAST, const v4i* cur, const v4i* nxt, const v4i* b, int rb_stride, int i_stride, v16i* acc, auto between) {
        auto operand = [&](int i) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) bq[i % PF][rb] = b[(rb * rb_stride + i * i_stride) * 64 + lane];
        };
#pragma unroll
        for (int i = 0; i < KS; ++i) {
            constexpr int S0 = decltype(SLOT0)::value;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) acc[rb] = mfma32(ring[(S0 + i) % RING], bq[i % PF][rb], acc[rb]);
            if (i + RING < KS) ring[(S0 + i) % RING] = cur[(i + RING) * 64];
            else if (!decltype(LAST)::value) ring[(S0 + i) % RING] = nxt[(i + RING - KS) * 64];
            if (i + PF < KS) operand(i + PF);
            between(i);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using Even = std::integral_constant<int, 0>;
    using Odd = std::integral_constant<int, SLOT_ODD>;
    using More = std::false_type;
    auto nothing = [](int) {};
    auto start = [&](v16i* acc, int off) {                             // accumulators start at -zp * colsum
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
            const int4 t4 = *(const int4*)(prmi + off + qd * 8 + g * 4);
            acc[0][qd * 4 + 0] = t4.x; acc[0][qd * 4 + 1] = t4.y; acc[0][qd * 4 + 2] = t4.z; acc[0][qd * 4 + 3] = t4.w;
        }
#pragma unroll
        for (int rb = 1; rb < RB; ++rb) acc[rb] = acc[0];
    };
    if (pack) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) actf[(rb * KS + wave) * 64 + lane] = expand_codes(pc[rb], pack, g);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                   // the direct loads have landed
    __syncthreads();                                                  // staged codes, parameters and table visible
    // Shortcut of the first residual, in flight during the projection (requested before the barrier, its loads waited for the
    // pixel index behind the whole ring, one more round trip: C = 384, 96 windows, a pair of blocks 80.8 -> 76.2 us, with h no
    // longer parked on 32-row tiles).  Rows without a pixel are not stored: any values do, except for taps.
    float4 sc[RB][4];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        if (WHOLE) pix[rb] = whole_pix[min(group * 32 + j, TOK - 1)];
        pix[rb] = valid[rb] ? pix[rb] : -1;
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
            const float4 v = *(const float4*)(A.x + (size_t)max(pix[rb], 0) * C + nb * 32 + qd * 8 + g * 4);
            sc[rb][qd] = !TAPS || pix[rb] >= 0 ? v : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
    float h[RB][16];
    {   // output projection + first residual
        v16i acc[RB];
        start(acc, PR::P_NC + nb * 32);
        request(actf, KS, 1);
        run(Even(), More(), wproj, w1_of(0), actf, KS, 1, acc, nothing);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {
                const int n0 = nb * 32 + qd * 8 + g * 4;
                const float4 m = *(const float4*)(prm + PR::P_M + n0), bs = *(const float4*)(prm + PR::P_B + n0);
                h[rb][qd * 4 + 0] = fmaf(sum_value<SHORT>(acc[rb][qd * 4 + 0]), m.x, bs.x) + sc[rb][qd].x;
                h[rb][qd * 4 + 1] = fmaf(sum_value<SHORT>(acc[rb][qd * 4 + 1]), m.y, bs.y) + sc[rb][qd].y;
                h[rb][qd * 4 + 2] = fmaf(sum_value<SHORT>(acc[rb][qd * 4 + 2]), m.z, bs.z) + sc[rb][qd].z;
                h[rb][qd * 4 + 3] = fmaf(sum_value<SHORT>(acc[rb][qd * 4 + 3]), m.w, bs.w) + sc[rb][qd].w;
                if (PARK_H && pix[rb] >= 0)
                    *(float4*)(A.y + (size_t)pix[rb] * C + n0) = make_float4(h[rb][qd * 4], h[rb][qd * 4 + 1], h[rb][qd * 4 + 2], h[rb][qd * 4 + 3]);
                if (TAPS && valid[rb]) {
                    if (A.tap_acc_proj) *(int4*)(A.tap_acc_proj + canon[rb] * C + n0) = make_int4(sum_int<SHORT>(acc[rb][qd * 4]), sum_int<SHORT>(acc[rb][qd * 4 + 1]), sum_int<SHORT>(acc[rb][qd * 4 + 2]), sum_int<SHORT>(acc[rb][qd * 4 + 3]));
                    if (A.tap_h) *(float4*)(A.tap_h + canon[rb] * C + n0) = make_float4(h[rb][qd * 4], h[rb][qd * 4 + 1], h[rb][qd * 4 + 2], h[rb][qd * 4 + 3]);
                }
            }
    }
    {   // LN2: binary64 partial sums per (wave, token) through LDS, then normalise and quantize
        float mean[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            double s = 0.0;
#pragma unroll
            for (int r = 0; r < 16; r += 4) s += sum4(h[rb][r], h[rb][r + 1], h[rb][r + 2], h[rb][r + 3]);
            s = half_sum(s);
            if (g == 0) part[0][wave][rb * 32 + j] = s;
        }
        __syncthreads();                                              // also: every wave is done reading the attention codes
        // sum of a row's partials: with an even number of waves each half of the lanes takes every second one, read together
        auto total = [&](int which, int rb) {
            constexpr bool HALVES = NH % 2 == 0;
            constexpr int N = HALVES ? NH / 2 : NH;
            double v[N];
#pragma unroll
            for (int k = 0; k < N; ++k) v[k] = part[which][HALVES ? 2 * k + g : k][rb * 32 + j];
#pragma unroll
            for (int d = 1; d < N; d *= 2)
#pragma unroll
                for (int k = 0; k + d < N; k += 2 * d) v[k] += v[k + d];
            return HALVES ? half_sum(v[0]) : v[0];
        };
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) mean[rb] = ln_mean(total(0, rb), C);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            double q = 0.0;
#pragma unroll
            for (int r = 0; r < 16; r += 4) q += centred4<false>(h[rb][r], h[rb][r + 1], h[rb][r + 2], h[rb][r + 3], mean[rb]);
            q = half_sum(q);
            if (g == 0) part[1][wave][rb * 32 + j] = q;
        }
        __syncthreads();
        const QDev qa = in_vgpr(A.q_fc1in[branch]);
        float rstd[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) rstd[rb] = ln_rstd(total(1, rb), C, A.eps);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            int wd[4];
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {
                const int n0 = nb * 32 + qd * 8 + g * 4;
                const float4 gm = *(const float4*)(prm + PR::LN_G + n0), bt = *(const float4*)(prm + PR::LN_B + n0);
                wd[qd] = pack4(quant_code(fmaf((h[rb][qd * 4 + 0] - mean[rb]) * rstd[rb], gm.x, bt.x), qa),
                               quant_code(fmaf((h[rb][qd * 4 + 1] - mean[rb]) * rstd[rb], gm.y, bt.y), qa),
                               quant_code(fmaf((h[rb][qd * 4 + 2] - mean[rb]) * rstd[rb], gm.z, bt.z), qa),
                               quant_code(fmaf((h[rb][qd * 4 + 3] - mean[rb]) * rstd[rb], gm.w, bt.w), qa));
                if (TAPS && valid[rb] && A.tap_a2) *(int*)(A.tap_a2 + canon[rb] * C + n0) = wd[qd];
            }
            actf[(rb * KS + nb) * 64 + lane] = (v4i){wd[0], wd[1], wd[2], wd[3]};   // k slab nb, byte r = channel 32nb + mfma_row(r,g)
        }
    }
    __syncthreads();
    v16i acc2[RB];
    start(acc2, PR::F2_NC + nb * 32);
    QDev qg;
    GeluIndex gi;
    if constexpr (SHORT) gi = in_vgpr(A.step_index[branch]); else qg = in_vgpr(A.q_fc2in[branch]);
    // GELU + quantize of four of the FC1 sums of hidden block ch*NH + wave, and the block's codes -> LDS buffer ch & 1
    int wd[RB][4];
    auto gelu_part = [&](int ch, int rb, int qd, const v16i* acc) {
        const int n0 = (ch * NH + wave) * 32 + qd * 8 + g * 4;
        const float4 m = *(const float4*)(prm + PR::F1_M + n0), bs = *(const float4*)(prm + PR::F1_B + n0);
        std::conditional_t<SHORT, GeluStepPart, GeluPart> p;
        p.xs[0] = fmaf(sum_value<SHORT>(acc[rb][qd * 4 + 0]), m.x, bs.x); p.xs[1] = fmaf(sum_value<SHORT>(acc[rb][qd * 4 + 1]), m.y, bs.y);
        p.xs[2] = fmaf(sum_value<SHORT>(acc[rb][qd * 4 + 2]), m.z, bs.z); p.xs[3] = fmaf(sum_value<SHORT>(acc[rb][qd * 4 + 3]), m.w, bs.w);
        if constexpr (SHORT) { gelu_begin(p, (const GeluStep*)gtab, gi); wd[rb][qd] = gelu_end(p); }
        else { gelu_begin(p, gtab); wd[rb][qd] = gelu_end(p, qg); }
        if (TAPS && valid[rb]) {
            if (A.tap_acc_fc1) *(int4*)(A.tap_acc_fc1 + canon[rb] * F + n0) = make_int4(sum_int<SHORT>(acc[rb][qd * 4]), sum_int<SHORT>(acc[rb][qd * 4 + 1]), sum_int<SHORT>(acc[rb][qd * 4 + 2]), sum_int<SHORT>(acc[rb][qd * 4 + 3]));
            if (A.tap_g) *(int*)(A.tap_g + canon[rb] * F + n0) = wd[rb][qd];
        }
    };
    auto gelu_store = [&](int ch) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) gs[ch & 1][(wave * RB + rb) * 64 + lane] = (v4i){wd[rb][0], wd[rb][1], wd[rb][2], wd[rb][3]};
    };
    {   // chunk 0: FC1 + GELU
        v16i acc[RB];
        start(acc, PR::F1_NC + wave * 32);
        request(actf, KS, 1);
        run(Odd(), More(), w1_of(0), w1_of(1), actf, KS, 1, acc, nothing);
        request(actf, KS, 1);
#pragma unroll
        for (int u = 0; u < 4 * RB; ++u) gelu_part(0, u / 4, u % 4, acc);
        gelu_store(0);
    }
    __syncthreads();                                                  // chunk 0 of the hidden codes complete
#pragma unroll 1
    for (int ch = 1; ch < 4; ++ch) {
        v16i acc[RB];
        start(acc, PR::F1_NC + (ch * NH + wave) * 32);
        run(Even(), More(), w1_of(ch), w2_of(ch - 1), actf, KS, 1, acc, nothing);                          // FC1 of chunk ch
        request(gs[(ch - 1) & 1], 1, RB);
        run(Odd(), More(), w2_of(ch - 1), ch < 3 ? w1_of(ch + 1) : w2_of(3), gs[(ch - 1) & 1], 1, RB, acc2,   // FC2 of chunk ch-1, and
            [&](int i) {                                                                      // between its steps ...
#pragma unroll
                for (int u = 0; u < 4 * RB; ++u)
                    if (((u + 1) * KS + 4 * RB - 1) / (4 * RB) - 1 == i) gelu_part(ch, u / 4, u % 4, acc);   // ... GELU of chunk ch
            });
        gelu_store(ch);
        if (ch < 3) request(actf, KS, 1);
        __syncthreads();                                              // chunk ch complete, chunk ch-1 no longer read
    }
    if (PARK_H) {                                                     // the parked h travels under the last products
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {
                const float4 v = *(const float4*)(A.y + (size_t)max(pix[rb], 0) * C + nb * 32 + qd * 8 + g * 4);
                h[rb][qd * 4] = v.x; h[rb][qd * 4 + 1] = v.y; h[rb][qd * 4 + 2] = v.z; h[rb][qd * 4 + 3] = v.w;
            }
    }
    request(gs[1], 1, RB);
    run(Even(), std::true_type(), w2_of(3), nullptr, gs[1], 1, RB, acc2, nothing);                     // FC2 of the last chunk
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {   // second residual + scatter
            const int n0 = nb * 32 + qd * 8 + g * 4;
            const float4 m = *(const float4*)(prm + PR::F2_M + n0), bs = *(const float4*)(prm + PR::F2_B + n0);
            const float4 hh = make_float4(h[rb][qd * 4], h[rb][qd * 4 + 1], h[rb][qd * 4 + 2], h[rb][qd * 4 + 3]);
            float4 o4 = make_float4(fmaf((float)acc2[rb][qd * 4 + 0], m.x, bs.x) + hh.x, fmaf((float)acc2[rb][qd * 4 + 1], m.y, bs.y) + hh.y,
                                    fmaf((float)acc2[rb][qd * 4 + 2], m.z, bs.z) + hh.z, fmaf((float)acc2[rb][qd * 4 + 3], m.w, bs.w) + hh.w);
            if (pix[rb] >= 0) *(float4*)(A.y + (size_t)pix[rb] * C + n0) = o4;
            if (TAPS && valid[rb]) {
                if (A.tap_acc_fc2) *(int4*)(A.tap_acc_fc2 + canon[rb] * C + n0) = make_int4(acc2[rb][qd * 4], acc2[rb][qd * 4 + 1], acc2[rb][qd * 4 + 2], acc2[rb][qd * 4 + 3]);
                if (A.tap_y) *(float4*)(A.tap_y + canon[rb] * C + n0) = o4;
            }
        }
}

template <int NH, int RB, bool TAPS, bool SHORT>
__global__ __launch_bounds__(NH * 64) __attribute__((amdgpu_waves_per_eu(tok_waves_per_eu(NH)))) void token_kernel(Geom G, TokArgs A)
{
    if (NH == 12 || G.rows_total <= 256 * 32) touch_arguments<sizeof(Geom) + sizeof(TokArgs)>();   // about one workgroup a CU
    __shared__ TokLds<NH, RB, 1, SHORT> lds;
    token_half<NH, RB, TAPS, SHORT, 1, false>(G, A, lds, 0, nullptr, nullptr);
}

// ------------------------------------------------------------------ a whole block on small maps
// One workgroup per window runs both halves of the block: the window kernel's form of pairs of waves, by roles, then two token kernels of
// one row block side by side for the window's 32 and 17 rows, each wave one of a tile's channel blocks.  What the halves hand on stays in
// LDS.  The second half's parameters and table are requested ahead of LN1, but behind the first half's, and the barrier in front of LN1
// waits for them, so their way is not hidden.  The compiler keeps the branch, which is handed on by reference behind a divergent copy, in
// vector registers, and what it chooses comes by vector loads, most followed by a wait for all loads: 61 vector loads and 18 such waits in
// the form that ranks its window at C = 96.  Bound: the chain of dependent steps, these waits among them, of a workgroup that has a CU to
// itself or shares it with one other.  The codes of the attention take the room of LN1's and the hidden codes that of the pairs' exchange,
// so that at C = 96 and 128 two workgroups fit a CU, with 128 registers (one spilled at C = 128).  (The first weights of the projection
// requested ahead of the attention, with those waits in place: nothing.)  Window and token kernel -> this one, one block on 56 x 56 x 96
// 17.0 -> 16.1 us, two on 256 windows 37.1 -> 32.9, at C = 192 57.9 -> 50.3; more beside whole_block(), which draws the lines.
constexpr int whole_waves_per_eu(int NH) { return NH == 6 ? 3 : 4; }
template <int NH, bool SCORED>
__global__ __launch_bounds__(NH * 2 * 64) __attribute__((amdgpu_waves_per_eu(whole_waves_per_eu(NH)))) void block_kernel(Geom G, WinArgs W, TokArgs T)
{
    touch_arguments<sizeof(Geom) + sizeof(WinArgs) + sizeof(TokArgs)>();
    __shared__ TokLds<NH, 1, 2, true> lds;
    __shared__ v4i exchange[NH * 5 * 64];                              // of the pairs, then the hidden codes of both tiles
    __shared__ int pix[64];
    static_assert(NH * 5 >= 2 * 2 * NH, "room for two buffers of two tiles");
    const int lane = threadIdx.x & 63, swave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int branch;
    const bool computed = window_half<NH, false, SCORED, 1, 2, false, true, false, true>(G, W, branch, WholeLds{lds.actf[0], exchange, pix}, [&] {
        token_stage<2 * NH, TokPrm<NH * 32>::WORDS>(T.params[branch], (const float4*)T.steps[branch], T.step_pieces[branch], lds.prm, lds.gtab, swave, lane);
    });
    if (!computed) return;
    token_half<NH, 1, false, true, 2, true>(G, T, lds, branch, pix, (v4i (*)[2][NH * 64])exchange);
}

// ------------------------------------------------------------------ launchers
// From C = 384 a window is taken by 1024 threads (256 threads -> 1024, launch to launch on fresh maps).  Raw score: equal where
// the launch itself is what takes the time (24 windows at C = 768 6.5 us both), better or equal beyond (384 windows at 768 12.5 ->
// 11.7, 3200 at 384 41.8 -> 39.1, 900 at 1024 30.8 -> 30.5).  With the scoring LayerNorm the window's arithmetic is spread wider
// (24 windows at 768 11.0 -> 7.5, 100 at 1024 14.1 -> 9.3, 900 at 384 17.6 -> 16.6), until the map no longer fits the chip in
// about one round and the waiting of the larger workgroups costs more (1600 windows at 384 28.4 -> 28.6, 1444 at 512 34.0 ->
// 36.1, 900 at 768 30.3 -> 36.2, 900 at 1024 39.1 -> 45.0): the line is drawn at windows times channels.
constexpr long long SCORE_WIDE_LN_MAX = 512 * 1024;
template <int LPT, int NV>
static void launch_score_t(const Geom& G, const float* x, int mode, float eps, const float* gm, const float* bt,
                           double* scores, hipStream_t st)
{
    constexpr bool WIDE = LPT * NV * 4 >= 384;
    if (WIDE && (mode == 0 || (long long)G.B * G.nW * G.C <= SCORE_WIDE_LN_MAX))
        hipLaunchKernelGGL((score_kernel<LPT, NV, WIDE ? 1024 : 256>), dim3(G.B * G.nW), dim3(WIDE ? 1024 : 256), 0, st, G, x, mode, eps, gm, bt, scores);
    else
        hipLaunchKernelGGL((score_kernel<LPT, NV, 256>), dim3(G.B * G.nW), dim3(256), 0, st, G, x, mode, eps, gm, bt, scores);
}
template <int LPT, int NV>
static void launch_ln_t(const Geom& G, const LnArgs& A, bool gather, hipStream_t st)
{
    constexpr int TP = 256 / LPT;
    if (G.rows_total == 0) return;
    dim3 grid((G.rows_total + TP - 1) / TP);
    if (gather) hipLaunchKernelGGL((ln_quant_kernel<LPT, NV, true>), grid, dim3(256), 0, st, G, A);
    else hipLaunchKernelGGL((ln_quant_kernel<LPT, NV, false>), grid, dim3(256), 0, st, G, A);
}

#define MIXAQ_DISPATCH_C(C, CALL)                                             \
    switch (C) {                                                              \
        case 96: CALL(8, 3); break;                                           \
        case 128: CALL(8, 4); break;                                          \
        case 192: CALL(16, 3); break;                                         \
        case 256: CALL(16, 4); break;                                         \
        case 384: CALL(32, 3); break;                                         \
        case 512: CALL(32, 4); break;                                         \
        case 768: CALL(64, 3); break;                                         \
        case 1024: CALL(64, 4); break;                                        \
        default: return false;                                                \
    }

bool channels_supported(int C)
{
    return C == 96 || C == 128 || C == 192 || C == 256 || C == 384 || C == 512 || C == 768 || C == 1024;
}

bool launch_score(const Geom& G, const float* x, int mode, float eps, const float* gm, const float* bt, double* scores,
                  hipStream_t st)
{
#define CALL(L, N) launch_score_t<L, N>(G, x, mode, eps, gm, bt, scores, st)
    MIXAQ_DISPATCH_C(G.C, CALL)
#undef CALL
    return true;
}

void launch_bypass(const Geom& G, const int* perm, const float* x, float* y, hipStream_t st)
{
    const int n_pruned = G.nW - G.k_hi - G.k_lo;
    if (n_pruned > 0) hipLaunchKernelGGL(bypass_kernel, dim3(G.B * n_pruned), dim3(256), 0, st, G, perm, x, y);
}

void launch_select(const double* scores, int B, int nW, int reverse, int* perm, hipStream_t st)
{
    hipLaunchKernelGGL(select_rank_kernel, dim3((nW + RANK_WPB - 1) / RANK_WPB, B), dim3(256), (size_t)nW * 8, st, scores, nW, reverse,
                       perm);
}

bool launch_ln_quant(const Geom& G, const LnArgs& A, bool gather, hipStream_t st)
{
#define CALL(L, N) launch_ln_t<L, N>(G, A, gather, st)
    MIXAQ_DISPATCH_C(G.C, CALL)
#undef CALL
    return true;
}

// FC1 on 128 x 128 tiles, whose epilogue is the longest, takes one slab a stage: 48 KB, three workgroups on a CU, one's GELU beside the others'
// products (T = 3696 67 -> 64, 3552 82 -> 74); the others two slabs, two workgroups.
template <int EPI, int WY, int WX, int RB, int NBW, int KSL, int S, int WPE>
static void launch_ring(const Geom& G, const GemmArgs& A, hipStream_t st)
{
    constexpr int LDS = (WY * RB + WX * NBW) * KSL * S * 1024 + WX * NBW * 768 + (EPI == EPI_FC1 ? GELU_STEP_PIECES * 1024 : 16);
    constexpr int PER_CU = std::min(160 * 1024 / LDS, 4 * WPE / (WY * WX));                  // more tiles than the chip holds at once: a workgroup takes several
    const int tiles = (G.rows_total / (WY * RB * 32)) * (A.N / (WX * NBW * 32));
    const dim3 grid(std::min((tiles + 7) / 8 * 8, CUS * PER_CU)), block(WY * WX * 64);
    if constexpr (EPI == EPI_FC1)
        if (A.steps[0]) {
            hipLaunchKernelGGL((gemm_ring_kernel<EPI, WY, WX, RB, NBW, KSL, S, WPE, true>), grid, block, 0, st, G, A);
            return;
        }
    hipLaunchKernelGGL((gemm_ring_kernel<EPI, WY, WX, RB, NBW, KSL, S, WPE, false>), grid, block, 0, st, G, A);
}
template <int EPI>
static void launch_few(const Geom& G, const GemmArgs& A, hipStream_t st)
{
    constexpr int WIDER = EPI == EPI_FC2 ? 4 : 1;
    const dim3 grid(G.rows_total / 32 * (A.N / 32)), block(512);
    if (A.K == 512 * WIDER) hipLaunchKernelGGL((gemm_few_kernel<EPI, 2 * WIDER>), grid, block, 0, st, G, A);
    else if (A.K == 768 * WIDER) hipLaunchKernelGGL((gemm_few_kernel<EPI, 3 * WIDER>), grid, block, 0, st, G, A);
    else hipLaunchKernelGGL((gemm_few_kernel<EPI, 4 * WIDER>), grid, block, 0, st, G, A);
}
template <int EPI>
static void launch_gemm_e(const Geom& G, const GemmArgs& A0, hipStream_t st)
{
    GemmArgs A = A0;
    if (G.rows_total == 0) return;
    switch (product_form(EPI, G.rows_total, A.N, A.K)) {
        case FEW:
            if constexpr (EPI == EPI_PROJ || EPI == EPI_FC2) launch_few<EPI>(G, A, st);
            return;
        case RING64:
            if constexpr (EPI == EPI_FC1)
                if (fc1_ring_of_four(G.rows_total, A.N)) { launch_ring<EPI, 2, 2, 1, 1, 2, 3, 4>(G, A, st); return; }
            launch_ring<EPI, 2, 2, 1, 1, 4, 4, 2>(G, A, st);
            return;
        case RING128:
            if constexpr (EPI == EPI_FC1) launch_ring<EPI, 2, 2, 2, 2, 1, 4, 3>(G, A, st);
            else launch_ring<EPI, 2, 2, 2, 2, 2, 4, 2>(G, A, st);
            return;
        case TILE: break;
    }
    // the activation tile through LDS, output blocks over the waves and, while the grid is small, in groups over workgroups; a narrow layer
    // on few rows in 32-row tiles: twice the workgroups
    const int tiles = G.rows_total / ROW_TILE, NB = A.N / 32;
    const bool half = EPI == EPI_FC2 && tiles <= 32 && A.K > 384 && A.K <= 1024;
    const int nt = half ? G.rows_total / 32 : tiles;
    const int groups = std::max(1, std::min((NB + 3) / 4, (512 + nt - 1) / nt));
    A.nb_per_block = ((NB + groups - 1) / groups + 3) / 4 * 4;
    const dim3 grid(nt, (NB + A.nb_per_block - 1) / A.nb_per_block);
#define GEMM_CASE(KMAX, RT, D) hipLaunchKernelGGL((gemm_tile_kernel<EPI, KMAX, RT, D>), grid, dim3(256), 0, st, G, A)
    if constexpr (EPI == EPI_FC2) {                                   // only FC2 has another K than C, up to 7 * 192 here
        if (A.K > 1024) { GEMM_CASE(1344, 64, 12); return; }
        if (half) { GEMM_CASE(1024, 32, 12); return; }
        if (A.K > 384) { GEMM_CASE(1024, 64, 12); return; }
    }
    GEMM_CASE(384, 64, 6);
#undef GEMM_CASE
}

void launch_gemm(const Geom& G, const GemmArgs& A, int epi, hipStream_t st)
{
    switch (epi) {
        case EPI_QKV: launch_gemm_e<EPI_QKV>(G, A, st); break;
        case EPI_PROJ: launch_gemm_e<EPI_PROJ>(G, A, st); break;
        case EPI_FC1: launch_gemm_e<EPI_FC1>(G, A, st); break;
        default: launch_gemm_e<EPI_FC2>(G, A, st); break;
    }
}

// the window kernel (gather + LN1 + QKV + attention) and the token kernel (proj + LN2 + FFN + scatter) are chosen separately
bool fused_token_supported(int C, int mlp_ratio) { return (C == 96 || C == 128 || C == 192 || C == 256 || C == 384) && mlp_ratio == 4; }

// Forms of the window kernel by the number of windows.  One wave per head has the fewest instructions per window; a pair of waves per head
// has the shorter chain of dependent steps at 15 % more vector and 80 % more scalar instructions; two workgroups per window, each
// with half its heads in pairs (both gather and normalize the whole window), put fewer waves side by side on a SIMD.  Measured
// as two blocks on one map, us, in the order single / pair / split (three sets of handles in turn):
//   C = 96   66 windows 40 / 34   228 46 / 39   260 47 / 44   360 52 / 49   506 56 / 53   528 60 / 63   600 62 / 64; each of two chains (six
//            blocks): 260 172 / 160   400 196 / 189   504 219 / 212   600 239 / 242   704 263 / 275
//   C = 128  66 40 / 36 / 34   126 40 / 36 / 35   140 41 / 37 / 38   256 46 / 41 / 42   266 49 / 48 / 46   378 55 / 54 / 52   396 56 / 54 / 56
//            506 62 / 60 / 63   528 68 / 71 / 69; each of two chains: 112 (twelve blocks) 276 / 253 / 246   260 184 / 177 / 169   400 218 / 215 / 219
//            504 254 / 256 / 261   600 291 / 301 / 307
//   C = 192  66 51 / 52 / 44   126 52 / 53 / 46   140 52 / 54 / 52   256 64 / 65 / 63   266 73 / 71 / 75   360 87 / 86 / 88   506 102 / 101 / 112
//            576 127 / 127 / 135; each of two chains: 77 182 / 183 / 166   112 188 / 188 / 186   126 190 / 191 / 191   144 202 / 194 / 211
//            198 240 / 231 / 236   228 257 / 253 / 258   260 274 / 282 / 287   400 377 / 406 / 418
//   C = 384  single / split: 66 80 / 72   126 82 / 75   140 84 / 97   187 117 / 130; each of two chains: 50 251 / 227   70 260 / 240   77 263 / 259
//            91 280 / 292   112 322 / 339
// C = 96 and 128: pairs while a CU has no more than two of their workgroups, and at C = 128 split wherever that leaves fewer waves on
// the fullest CU.  C = 192: split, then pairs, while a CU has no more than two of their workgroups, both chains counted, as it has
// no room for a third.  C = 384: split while a CU has one (of two chains a few more: they are seldom in the same kernel).  Pruned windows
// count where their workgroups stand in the way of others, but not at C = 96 (461 of 576 computed: single 57, pair 56; 470 of 784 61, 59) and
// not beside a second chain at C = 384 (58 of 96, six blocks: single 252, split 233; 77 of 96 258 both); elsewhere counting the
// computed ones only measured slower (C = 384, 127 of 182 computed: 84 -> 90; 192, 240 of 300: 69 -> 71; 128, 461 of 576: 60 -> 62).
// C = 256 always split: sixteen waves of one workgroup, or eight of twice the registers, leave a CU half empty, three workgroups of
// eight fill it (6 windows: 62.8 -> 51.4 us the pair, 300: 106 -> 95, 1444: 351 -> 335, 2750: 680 -> 654).
enum WindowForm { SINGLE, PAIR, SPLIT };
// of a launch over `windows`, `computed` of them not pruned, beside another one like it where the stage runs as two chains
static WindowForm window_form(int heads, int windows, int computed, int chains)
{
    auto per_cu = [](int workgroups) { return (workgroups + CUS - 1) / CUS; };
    switch (heads) {
        case 3: return computed <= 2 * CUS ? PAIR : SINGLE;
        case 4: return windows > 2 * CUS ? SINGLE : 4 * per_cu(2 * windows) < 8 * per_cu(windows) ? SPLIT : PAIR;
        case 6: return windows * chains <= CUS ? SPLIT : windows * chains <= 2 * CUS ? PAIR : SINGLE;
        case 12: return windows <= CUS / 2 && (chains == 1 || computed <= 80) ? SPLIT : SINGLE;
        default: return SPLIT;
    }
}
// C = 96 beside a second chain: the forms that leave it room (see win_roles): pairs, and one wave per head while the launch is more than three
// and no more than five windows a CU.  There the two chains fall into step such that one's windows meet the tail of the other's token
// kernel, and five workgroups of three waves on a CU, all of the launch at once, keep out of it better than six.  Five waves per SIMD ->
// four, us, windows of both chains, two blocks / six:   1624 108.4 -> 108.0 / 276 -> 270   1740 112.8 -> 111.5 / 291 -> 282   1860 119.4 ->
// 117.1 / 305 -> 295   2046 125.8 -> 125.7 / 327 -> 324   2244 132.9 -> 133.1 / 351 -> 343   2520 144.4 -> 144.5 / 385 -> 385.  Outside of
// that, with the token kernel at four workgroups a CU instead of five:   1260 95.7 -> 97.9 / 237 -> 243   1428 103.4 -> 105.5 / 271 -> 268 |
// 2856 172.8 -> 170.2 / 473 -> 476   4 x 1392 315.9 -> 318.4 / 864 -> 870
static bool window_beside(WindowForm form, int windows, int chains) { return chains > 1 && (form == PAIR || (windows > 3 * CUS && windows <= 5 * CUS)); }
void launch_window(const Geom& G, const WinArgs& A, int chains, hipStream_t st)
{
    // every window gets a workgroup: with scores it finds its own rank (and may turn out pruned), otherwise
    // the computed slots come first and the pruned windows of the list after them
    const int n_wg = G.B * G.nW;
    if (n_wg == 0) return;
    // Wide blocks: LN1 by a kernel of its own, then the heads of a window over several workgroups: pairs of waves while each workgroup has a
    // CU to itself, one wave per head beyond, whose weights pass the L1 once instead of one and a half times.  LN1 and window kernel, us, pairs /
    // four heads a workgroup of one wave each / eight:   C = 512   49 windows 14.0 / 15.7 / 17.6   64 14.9 / 16.9 / 18.3 | 100 22.7 / 22.2 / 20.7
    //   270 49 / 43 / 45   784 115 / 95 / 97      C = 768   35 16.6 / 18.4 / 26.8   42 18.0 / 19.7 / 29.0 | 48 24.9 / 23.8 / 30.3   140 48 / 45 / 50
    //   400 112 / 102 / 98      C = 1024   25 18.4 / 29.7 / 24.4   30 19.6 / 32.0 / 25.2 | 42 29.8 / 38.1 / 27.9   100 55 / 57 / 48   288 120 / 110 / 111
#define WIN_LAUNCH(ARGS, SCORED, NH, HG, QS, CODES, BESIDE)   /* taps: one chain */                                        \
    if (ARGS.taps && ARGS.magic_sums) hipLaunchKernelGGL((window_kernel<NH, true, SCORED, HG, QS, CODES, true, false>), grid, block, 0, st, G, ARGS);    \
    else if (ARGS.taps) hipLaunchKernelGGL((window_kernel<NH, true, SCORED, HG, QS, CODES, false, false>), grid, block, 0, st, G, ARGS);                 \
    else if (ARGS.magic_sums) hipLaunchKernelGGL((window_kernel<NH, false, SCORED, HG, QS, CODES, true, BESIDE>), grid, block, 0, st, G, ARGS);          \
    else hipLaunchKernelGGL((window_kernel<NH, false, SCORED, HG, QS, CODES, false, BESIDE>), grid, block, 0, st, G, ARGS);
#define WIDE_CASE(C_, LPT, NV, NH, HG, QS, WHEN)                                                                          \
    if (G.C == C_ && (WHEN)) {                                                                                                      \
        const dim3 lgrid(n_wg, 64 * LPT / 256);                                                                           \
        if (A.scores) hipLaunchKernelGGL((ln_window_kernel<LPT, NV, true>), lgrid, dim3(256), 0, st, G, A);               \
        else hipLaunchKernelGGL((ln_window_kernel<LPT, NV, false>), lgrid, dim3(256), 0, st, G, A);                       \
        if (G.n_slots == 0) return;                                                                                       \
        WinArgs W = A;                                                                                                    \
        if (A.scores) W.perm = A.perm_out;                                                                                \
        const dim3 grid(G.n_slots * HG), block(NH * QS * 64);                                                             \
        WIN_LAUNCH(W, false, NH, HG, QS, true, false)                                                                          \
        return;                                                                                                           \
    }
    const bool fits = G.n_slots * (G.heads / 4) <= CUS;
    WIDE_CASE(512, 32, 4, 4, 4, 2, fits)
    WIDE_CASE(768, 64, 3, 4, 6, 2, fits)
    WIDE_CASE(1024, 64, 4, 4, 8, 2, fits)
    WIDE_CASE(512, 32, 4, 4, 4, 1, true)
    WIDE_CASE(768, 64, 3, 4, 6, 1, true)
    WIDE_CASE(1024, 64, 4, 8, 4, 1, true)
#undef WIDE_CASE
#define WIN_CASE(NH, HG, QS, BESIDE)                                                                                      \
    {                                                                                                                     \
        const dim3 grid(HG > 1 ? (n_wg + 7) / 8 * 8 * HG : n_wg), block(NH * QS * 64);                                     \
        if (A.scores) {   /* no entry point takes scores and taps together */                                            \
            if (A.magic_sums) hipLaunchKernelGGL((window_kernel<NH, false, true, HG, QS, false, true, BESIDE>), grid, block, 0, st, G, A);       \
            else hipLaunchKernelGGL((window_kernel<NH, false, true, HG, QS, false, false, BESIDE>), grid, block, 0, st, G, A);                   \
        } else {                                                                                                          \
            WIN_LAUNCH(A, false, NH, HG, QS, false, BESIDE)                                                               \
        }                                                                                                                 \
    }                                                                                                                     \
    break
    const WindowForm form = window_form(G.C / 32, n_wg, G.n_slots, chains);
    switch (G.C / 32) {
        case 3:
            if (window_beside(form, n_wg, chains)) {
                if (form == PAIR) { WIN_CASE(3, 1, 2, true); }
                WIN_CASE(3, 1, 1, true);
            }
            if (form == PAIR) { WIN_CASE(3, 1, 2, false); }
            WIN_CASE(3, 1, 1, false);
        case 4:
            if (form == SPLIT) { WIN_CASE(2, 2, 2, false); }
            if (form == PAIR) { WIN_CASE(4, 1, 2, false); }
            WIN_CASE(4, 1, 1, false);
        case 6:
            if (form == SPLIT) { WIN_CASE(3, 2, 2, false); }
            if (form == PAIR) { WIN_CASE(6, 1, 2, false); }
            WIN_CASE(6, 1, 1, false);
        case 8: WIN_CASE(4, 2, 2, false);
        case 12:
            if (form == SPLIT) { WIN_CASE(6, 2, 2, false); }
            WIN_CASE(12, 1, 1, false);
        default: break;
    }
#undef WIN_CASE
#undef WIN_LAUNCH
}

// Rows per workgroup of the token kernel at C = 384.  A CU holds one workgroup of twelve waves, which takes 15 units of time for 64
// rows and 8 for 32, so the form is the one whose rounds over the CUs are shorter; two chains fill them together.  32 rows -> 64, us,
// two blocks on one map (three sets of handles in turn):
//   windows   66 72 -> 103   160 87 -> 114 | 170 121 -> 115   187 121 -> 117   260 157 -> 152   294 159 -> 161   330 164 -> 166 |
//             345 197 -> 228   384 203 -> 232   442 216 -> 241   486 226 -> 244 | 504 255 -> 247   513 286 -> 277   600 293 -> 291 |
//             704 338 -> 368   805 380 -> 403
// and six blocks, windows of each of two chains:  70 241 -> 331   96 299 -> 359   126 373 -> 407   150 393 -> 423   176 462 -> 503   198 537
// both   216 555 -> 598   240 592 -> 620 | 260 689 -> 667   280 700 -> 697   294 740 -> 724   322 784 -> 775 | 345 855 -> 870   360 892 -> 915
// | 400 999 -> 988   425 1031 -> 1032   600 1445 -> 1423 | 704 1698 -> 1717.
// While 64-row tiles of both chains are no more than the CUs the chains are seldom in this kernel together, and a long tile is
// the latency of one chain: 32 rows.  With fewer waves (C <= 256) the registers of a second row block cost more than its weights save.
static bool token_of_64_rows(int rows, int chains)
{
    const int all = rows * chains, tiles32 = all / 32, tiles64 = all / 64;
    if (chains > 1 && tiles64 <= CUS) return false;
    return 15 * ((tiles64 + CUS - 1) / CUS) < 8 * ((tiles32 + CUS - 1) / CUS);
}
void launch_token(const Geom& G, const TokArgs& A, int chains, hipStream_t st)
{
    if (G.rows_total == 0) return;
#define TOK_CASE(NH, RB)                                                                                                             \
    {                                                                                                                                \
        const dim3 grid(G.rows_total / (32 * RB)), block(NH * 64);                                                                   \
        if (A.short_forms && A.taps) hipLaunchKernelGGL((token_kernel<NH, RB, true, true>), grid, block, 0, st, G, A);                  \
        else if (A.short_forms) hipLaunchKernelGGL((token_kernel<NH, RB, false, true>), grid, block, 0, st, G, A);                      \
        else if (A.taps) hipLaunchKernelGGL((token_kernel<NH, RB, true, false>), grid, block, 0, st, G, A);                          \
        else hipLaunchKernelGGL((token_kernel<NH, RB, false, false>), grid, block, 0, st, G, A);                                     \
    }
    switch (G.C / 32) {
        case 3: TOK_CASE(3, 1) break;
        case 4: TOK_CASE(4, 1) break;
        case 6: TOK_CASE(6, 1) break;
        case 8: TOK_CASE(8, 1) break;
        default:
            if (token_of_64_rows(G.rows_total, chains)) TOK_CASE(12, 2)
            else TOK_CASE(12, 1)
    }
#undef TOK_CASE
}

bool launch_block(const Geom& G, const WinArgs& W, const TokArgs& T, int chains, hipStream_t st)
{
    const int windows = G.B * G.nW;
    if (W.taps || !W.magic_sums || !T.short_forms || chains > 1 || windows == 0 || !whole_block(G.C, windows, G.n_slots, W.scores != nullptr)) return false;
#define BLOCK_CASE(NH)                                                                                                                \
    if (W.scores) hipLaunchKernelGGL((block_kernel<NH, true>), dim3(windows), dim3(NH * 128), 0, st, G, W, T);                        \
    else hipLaunchKernelGGL((block_kernel<NH, false>), dim3(windows), dim3(NH * 128), 0, st, G, W, T);                                \
    return true
    switch (G.C / 32) {
        case 3: BLOCK_CASE(3);
        case 4: BLOCK_CASE(4);
        case 6: BLOCK_CASE(6);
        default: return false;
    }
#undef BLOCK_CASE
}

void launch_attn(const Geom& G, const AttnArgs& A, hipStream_t st)
{
    const int items = G.n_slots * G.heads;
    if (items == 0) return;
    hipLaunchKernelGGL(attn_kernel, dim3((items + 3) / 4), dim3(256), 0, st, G, A);
}

}  // namespace mixaq
