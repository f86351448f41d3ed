// Device-side building blocks shared by the gfx950 kernels of the Two-Branch
// Swin Block: the pinned binary32 arithmetic that decides integer codes, the
// int8 MFMA wrappers with their lane layouts, and the row-space bookkeeping.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "gelu_steps.h"
#include "ln_stats.h"

namespace mixaq {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int WS = 7;            // window side
constexpr int TOK = 49;          // tokens per window
constexpr int BIAS_QUADS = (TOK + 3) / 4;   // key quads of the bias table
constexpr int HD = 32;           // head dimension = one 32-wide MFMA block
constexpr int ROW_TILE = 64;     // rows per GEMM tile
constexpr int REGION_ALIGN = 128; // the branch regions of the row space are padded to this (the largest row tile of any kernel)
constexpr float LOG2E_F = 0x1.715476p+0f;
constexpr float MASK_VALUE = -100.0f;
constexpr float RND_MAGIC = 12582912.0f;          // 1.5 * 2^23: adding it rounds to an integer, ties to even

// One activation quantizer prepared for the device.  code = clamp(round-half-even(v*inv_s + zp)):
// u = fma(v, inv_s, MAGIC + zp) rounds the exact sum to an integer in one operation (ties to the
// even code), the clamp is taken on u, and the code is the low mantissa byte of u.
struct QDev {
    float inv_s;      // 1.0f / scale
    float magic;      // MAGIC + zp
    float lo, hi;     // MAGIC + qmin, MAGIC + qmax
    float scale;
    int   zp;
};

// Brings every 64-byte line of the kernel's arguments into the scalar cache, in one round trip.  They are written anew for every
// launch, so the first read of each line goes to memory, and a kernel that reads a field where it needs it meets such a
// round trip in the middle of its work, again and again: one block on 56 x 56 x 96 18.5 -> 17.8 us, 25 x 42 x 768 93.2 -> 91.3,
// backbone 613.5 -> 605.7.  For kernels of about one workgroup a CU; where others run meanwhile, the longer wait at the start costs
// as much as it saves (200 x 336 x 96 103.3 -> 104.2, 3 x 61 x 93 x 192 73.3 -> 74.2), under the first loads too (4 x 256 x 256 x 128
// 421 -> 433).
template <int BYTES>
__device__ __forceinline__ void touch_arguments()
{
    const auto* p = (const __attribute__((address_space(4))) int*)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr int LINES = (BYTES + 63) / 64;
    int any = p[0];
#pragma unroll
    for (int k = 1; k < LINES; ++k) any ^= p[k * 16];
    asm volatile("" :: "s"(any));
}

// returns the bit pattern of u; its low byte is the int8 code
__device__ __forceinline__ int quant_code(float v, const QDev& q)
{
    float u = fmaf(v, q.inv_s, q.magic);
    u = __builtin_amdgcn_fmed3f(u, q.lo, q.hi);
    return __float_as_int(u);
}
// the code as a sign-extended integer
__device__ __forceinline__ int code_value(int ubits) { return (int)(int8_t)(ubits & 0xff); }

// low bytes of four words -> one dword of int8 (byte k = code k)
__device__ __forceinline__ int pack4(int c0, int c1, int c2, int c3)
{
    int lo = __builtin_amdgcn_perm(c1, c0, 0x0c0c0400);
    int hi = __builtin_amdgcn_perm(c3, c2, 0x04000c0c);
    return lo | hi;
}

// An integer sum as a number.  MAGIC: the sum was started at SUM_MAGIC_BITS more, so that as a binary32 it IS 1.5 * 2^23 plus the sum
// while that stays inside +-2^22, and an exact subtraction (a fast instruction) replaces the conversion (a slow one).  Blocks whose
// weights and quantizers do not bound their sums so convert.  (Sums of q, k, v, P.V, the projection and FC1: 100 x 168 x 192 79.9 -> 78.9 us,
// 4 x 128 x 128 x 256 320.1 -> 316.7, 200 x 336 x 96 101.0 -> 100.2.  FC2's sums, sixteen of a tile's 112 and the widest ones, and those
// of Q K^T, whose accumulators start at an inline zero, are converted.)
constexpr int SUM_MAGIC_BITS = 0x4b400000;                        // of RND_MAGIC
template <bool MAGIC> __device__ __forceinline__ float sum_value(int a) { return MAGIC ? __int_as_float(a) - RND_MAGIC : (float)a; }
template <bool MAGIC> __device__ __forceinline__ int sum_int(int a) { return MAGIC ? a - SUM_MAGIC_BITS : a; }

// gfx950 runs binary32 multiply, add and fused multiply-add, 32-bit and / or / xor, right shifts, integer addition and moves at
// twice the rate of its other vector instructions (2.1 to 2.8 clocks a wave instead of 4.0 to 4.3, four waves per SIMD) as long
// as no operand is a scalar register; with one they take 4.0 to 4.3 as well, a literal constant costs nothing.  So what such an
// instruction uses over and over is held in vector registers (in_vgpr) or written as a literal.
__device__ __forceinline__ float in_vgpr(float v) { asm("" : "+v"(v)); return v; }
__device__ __forceinline__ QDev in_vgpr(QDev q) { q.inv_s = in_vgpr(q.inv_s); q.magic = in_vgpr(q.magic); return q; }

// y <- 2^y for N values, EXP2_FLOOR <= y <= 0: split by rounding, degree-5 polynomial on [-1/2, 1/2] (the coefficients are pinned),
// exact scaling by an addition to the exponent.  The definition holds y at EXP2_FLOOR from below; the caller does so where a logit
// can be that far below its row's maximum (AttnCore::floor).  The Horner steps of four values are one asm statement: the compiler
// would put the coefficients into scalar registers, and it separates dependent asm statements by a wait state.
constexpr float EXP2_FLOOR = -100.0f;
constexpr float EXP2_C5 = 0x1.5f48c8p-10f;                        // the leading coefficient, held in a vector register by the caller
#define MIXAQ_EXP2_BITS(C_) "i"(__builtin_bit_cast(int, C_))
#define MIXAQ_EXP2_REST MIXAQ_EXP2_BITS(0x1.3d107cp-7f), MIXAQ_EXP2_BITS(0x1.c6aeccp-5f), MIXAQ_EXP2_BITS(0x1.ebf906p-3f), \
                        MIXAQ_EXP2_BITS(0x1.62e430p-1f), MIXAQ_EXP2_BITS(0x1.000002p+0f)
template <int N>
__device__ __forceinline__ void exp2_pinned(float* y, float c5)
{
    static_assert(N == 4 || N == 1, "written out for these");
    float t[N], r[N], p[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        t[k] = y[k] + RND_MAGIC;                                  // the integer nearest to y (ties to even) in the low mantissa bits
        r[k] = y[k] - (t[k] - RND_MAGIC);
    }
    if constexpr (N == 4) {
#define MIXAQ_EXP2_STEP(I_) "v_fmaak_f32 %0, %0, %4, %" I_ "\n\tv_fmaak_f32 %1, %1, %5, %" I_ "\n\tv_fmaak_f32 %2, %2, %6, %" I_ "\n\tv_fmaak_f32 %3, %3, %7, %" I_ "\n\t"
        asm("v_fmaak_f32 %0, %13, %4, %8\n\tv_fmaak_f32 %1, %13, %5, %8\n\tv_fmaak_f32 %2, %13, %6, %8\n\tv_fmaak_f32 %3, %13, %7, %8\n\t"
            MIXAQ_EXP2_STEP("9") MIXAQ_EXP2_STEP("10") MIXAQ_EXP2_STEP("11") MIXAQ_EXP2_STEP("12")
            : "=&v"(p[0]), "=&v"(p[1]), "=&v"(p[2]), "=&v"(p[3])
            : "v"(r[0]), "v"(r[1]), "v"(r[2]), "v"(r[3]), MIXAQ_EXP2_REST, "v"(c5));
#undef MIXAQ_EXP2_STEP
    } else {
        asm("v_fmaak_f32 %0, %7, %1, %2\n\tv_fmaak_f32 %0, %0, %1, %3\n\tv_fmaak_f32 %0, %0, %1, %4\n\tv_fmaak_f32 %0, %0, %1, %5\n\tv_fmaak_f32 %0, %0, %1, %6"
            : "=&v"(p[0]) : "v"(r[0]), MIXAQ_EXP2_REST, "v"(c5));
    }
#pragma unroll
    for (int k = 0; k < N; ++k) y[k] = __int_as_float((int)((unsigned)__float_as_int(t[k]) << 23) + __float_as_int(p[k]));   // what MAGIC leaves in t is shifted out
}

// GELU(x) = max(x,0) - H(|x|), H(a) = a*Phi(-a) as a piecewise cubic: interval i of width
// 2^-GELU_LOG2K on [0,6) holds the cubic in d = fract(a * 2^GELU_LOG2K); beyond the last
// interval the argument is held at its end.  The coefficient table (one float4 per interval)
// lives in LDS; replicating it per lane group to spread the banks was measured and is no faster.
//
// The kernels evaluate it on SCALED values: xs = x * 2^GELU_LOG2K goes in, GELU(x) * 2^GELU_LOG2K
// comes out, with the table's coefficients scaled by the same power of two.  A power-of-two
// factor commutes with every binary32 rounding (no overflow or underflow is near), so each
// step is exactly 2^GELU_LOG2K times the unscaled step and the codes are the same bit for bit,
// provided the caller folds the factor into what surrounds the call: the dequantization that
// produces xs uses (2^GELU_LOG2K * m, 2^GELU_LOG2K * bias), the quantizer that consumes the
// result uses inv_s / 2^GELU_LOG2K.  This saves the multiply that would form the table index.
constexpr int GELU_LOG2K = 4;
constexpr int GELU_K = 6 << GELU_LOG2K;                       // intervals on [0,6)
constexpr int GELU_TAB = (GELU_K + 63) / 64 * 64;            // entries of the stored table (whole 1 KB pieces; zeros behind the intervals)
constexpr float GELU_SCALE = (float)(1 << GELU_LOG2K);
__device__ __forceinline__ void gelu_stage_table(float4* lds, const float4* tab, int tid, int nthreads)
{
    for (int e = tid; e < GELU_K; e += nthreads) lds[e] = tab[e];
}
// GELU and quantizer of four values in two halves: all four table reads are requested before the first is waited for (value after
// value, a wave alone waited four times: block of 56 x 56 x 96 18.9 -> 18.6 us, 2 x 50 x 84 x 384 293 -> 287.5, backbone 627 -> 621.5).
struct GeluPart { float xs[4], d[4]; float4 c[4]; };
__device__ __forceinline__ void gelu_begin(GeluPart& p, const float4* lds)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float u = fminf(fabsf(p.xs[e]), (float)GELU_K * 0x1.fffffep-1f);
        p.d[e] = __builtin_amdgcn_fractf(u);
        p.c[e] = lds[(int)u];
    }
}
__device__ __forceinline__ int gelu_end(const GeluPart& p, const QDev& q)
{
    int c[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float h = fmaf(p.c[e].w, p.d[e], p.c[e].z);
        h = fmaf(h, p.d[e], p.c[e].y);
        h = fmaf(h, p.d[e], p.c[e].x);
        c[e] = quant_code(fmaxf(p.xs[e], 0.0f) - h, q);
    }
    return pack4(c[0], c[1], c[2], c[3]);
}
// GELU and quantizer of four values by the table of steps (see gelu_steps.h), in two halves likewise.  The signs of the four values
// leave as bytes (0 or 0xff) by v_perm; a byte that loses one is at least one, so the subtraction stays inside it.  Per value
// and behind the dequantization four fused multiply-adds or ands of the fast kind and two others' share, where the cubic and the quantizer take
// seven slow and six fast ones; half the bytes out of LDS.  Cubic -> steps: one block on 56 x 56 x 96 17.64 -> 17.09 us, 200 x 336 x 96
// 103.7 -> 100.3, 8 x 200 x 336 x 96 660 -> 640, 100 x 168 x 192 85.1 -> 80.5, 3 x 61 x 93 x 192 72.8 -> 69.4, 2 x 50 x 84 x 384 279.4 ->
// 274.9, 4 x 256 x 256 x 128 437 -> 419, 4 x 128 x 128 x 256 334.6 -> 324.1, backbone 605 -> 595.
struct GeluStepPart { float xs[4]; GeluStep e[4]; };
__device__ __forceinline__ GeluIndex in_vgpr(GeluIndex i) { i.scale = in_vgpr(i.scale); i.offset = in_vgpr(i.offset); i.span = in_vgpr(i.span); return i; }
__device__ __forceinline__ void gelu_begin(GeluStepPart& p, const GeluStep* lds, const GeluIndex& ix)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float u = __builtin_amdgcn_fmed3f(fmaf(p.xs[e], ix.scale, ix.offset), 0.0f, 1.0f);   // one instruction
        const int at = __float_as_int(fmaf(u, ix.span, GELU_STEP_MAGIC)) & GELU_STEP_MASK;
        p.e[e] = *(const GeluStep*)((const char*)lds + at);
    }
}
__device__ __forceinline__ int gelu_end(const GeluStepPart& p)
{
    int v[4], f[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) { v[e] = __float_as_int(fmaf(p.xs[e], p.e[e].factor, p.e[e].addend)); f[e] = __float_as_int(p.e[e].factor); }
    const int below = __builtin_amdgcn_perm(v[1], v[0], 0x0c0c0b09) | __builtin_amdgcn_perm(v[3], v[2], 0x0b090c0c);
    return (pack4(f[0], f[1], f[2], f[3]) - (below & 0x01010101)) ^ (int)0x80808080;
}

// ---- packed sub-byte codes (tensors that cross a kernel boundary) ---------------------------------
// The attention-output codes of the LOW branch travel packed when its bit width allows: two codes per byte
// (widths 3 and 4) or four per byte (width 2), stored offset-binary (u = code + PACK_OFFSET, never negative) so
// that unpacking is a shift and a mask; the consumer removes the offset together with the zero point
// (sum_k u_k w_k - (zp + offset) * sum_k w_k).  The layout is chosen so that the producer (a lane of the window
// kernel holds, per query and head, the dims qd*8 + g*4 + e, qd = 0..3, e = 0..3, of its half g) packs without
// leaving the lane, and the consumer (a lane needs 16 consecutive channels) reads 8 contiguous bytes:
//   pack 1 (nibbles), row stride C/2, per head 16 bytes: dword p*2 + g (p = 0,1), byte e:
//       low nibble = u(dim p*16 + g*4 + e), high nibble = u(dim p*16 + 8 + g*4 + e)
//   pack 2 (two-bit fields), row stride C/4, per head 8 bytes: dword g, byte e, bits 2qd..2qd+1 = u(dim qd*8 + g*4 + e)
__host__ __device__ constexpr int pack_mode(int bits) { return bits <= 2 ? 2 : bits <= 4 ? 1 : 0; }
__host__ __device__ constexpr int pack_offset(int mode) { return mode == 2 ? 2 : mode == 1 ? 8 : 0; }

// A third form, for the kernels that multiply whole tiles of rows: MFMA operand fragments, one byte per code.  Rows in
// groups of 32, per group and slab of 32 channels 64 lanes x 16 bytes: lane = half * 32 + row, byte = channel of the half.
constexpr int PACK_FRAG = 3;
__device__ __forceinline__ size_t frag_offset(int row, int ch, int slabs)
{
    return (((size_t)(row >> 5) * slabs + (ch >> 5)) * 64 + ((ch & 31) >> 4) * 32 + (row & 31)) * 16 + (ch & 15);
}

// the same with the 32 channels of a slab in the order of MFMA result registers (byte r of a half: channel mfma_row(r, half))
__device__ __forceinline__ size_t frag_offset_reg(int row, int ch, int slabs)
{
    return (((size_t)(row >> 5) * slabs + (ch >> 5)) * 64 + ((ch >> 2) & 1) * 32 + (row & 31)) * 16 + ((ch & 31) >> 3) * 4 + (ch & 3);
}

// the 16 codes (offset-binary, one per byte, in channel order) of channels 32*ks + 16*half .. +15 of one packed row: the eight
// bytes that hold them, and the codes (apart, so that the load can be in flight)
__device__ __forceinline__ int2 packed_codes(const int8_t* packed_row, int mode, int ks, int half)
{
    return *(const int2*)(packed_row + (mode == 1 ? ks * 16 + half * 8 : ks * 8));
}
__device__ __forceinline__ v4i expand_codes(int2 w, int mode, int half)
{
    if (mode == 1) return (v4i){w.x & 0x0f0f0f0f, w.y & 0x0f0f0f0f, (w.x >> 4) & 0x0f0f0f0f, (w.y >> 4) & 0x0f0f0f0f};
    const int s = half * 4;
    return (v4i){(w.x >> s) & 0x03030303, (w.y >> s) & 0x03030303, (w.x >> (s + 2)) & 0x03030303, (w.y >> (s + 2)) & 0x03030303};
}

// ---- sums across lanes, in the vector unit (a __shfl goes through the LDS pipe: tens of clocks instead of a few) ----
// value of the lane in the same place of the other half of the wave, combined with the own one: r.lo + r.hi in both halves
__device__ __forceinline__ float half_max(float v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);   // {lo,lo}, {hi,hi}
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ int half_sum(int v)
{
    const auto r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    return (int)r[0] + (int)r[1];
}
__device__ __forceinline__ double half_sum(double v)
{
    const auto l = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(v), (unsigned)__double2loint(v), false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(v), (unsigned)__double2hiint(v), false, false);
    return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return v + __hiloint2double(hi, lo);
}
// butterfly over W = 2, 4, ... 64 consecutive lanes: inside a row of sixteen by DPP (quad permutes, then the mirrors: the
// partial sums are already equal inside a quad / half row), across rows by the row swaps
template <int W>
__device__ __forceinline__ double lanes_sum(double v)
{
    if (W >= 2) v = dpp_add<0xb1>(v);                            // quad_perm [1,0,3,2]
    if (W >= 4) v = dpp_add<0x4e>(v);                            // quad_perm [2,3,0,1]
    if (W >= 8) v = dpp_add<0x141>(v);                           // row_half_mirror
    if (W >= 16) v = dpp_add<0x140>(v);                          // row_mirror
    if (W >= 32) {
        const auto l = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(v), (unsigned)__double2loint(v), false, false);
        const auto h = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(v), (unsigned)__double2hiint(v), false, false);
        v = __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
    }
    if (W >= 64) v = half_sum(v);
    return v;
}

// D[32x32] += A[32 x 32k] * B[32k x 32]; lane l supplies row (A) / column (B) l%32 and
// the 16 k-values of half l/32; D register r of lane l is row (r/4)*8 + (l/32)*4 + r%4,
// column l%32.
__device__ __forceinline__ v16i mfma32(v4i a, v4i b, v16i c)
{
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
}
// row of the 32x32 result held in register r by a lane of half g
__device__ __forceinline__ int mfma_row(int r, int g) { return (r >> 2) * 8 + g * 4 + (r & 3); }

// n / d for 0 <= n < 2^31 and a divisor the host knows: a high product, an add and a shift in place of the some twenty-five
// instructions of a division
struct FastDiv {
    unsigned mul = 0, shift = 0;
    int d = 1;
    FastDiv() = default;
    explicit FastDiv(int divisor) : d(divisor)
    {
        while ((1u << shift) < (unsigned)divisor) ++shift;
        mul = (unsigned)(((1ull << 32) * ((1ull << shift) - (unsigned)divisor)) / (unsigned)divisor + 1);
    }
    __device__ __forceinline__ int operator()(int n) const { return (int)((__umulhi(mul, (unsigned)n) + (unsigned)n) >> shift); }
};

// Geometry of one forward call.  Rows of the gathered activation matrices: the
// high group of all images first (slot = b*k_hi + j), padded to a multiple of
// REGION_ALIGN, then the low group (slot = b*k_lo + j - k_hi).
struct Geom {
    int B, H, W, C, shift, heads;
    int Hp, Wp, nWc, nW;
    int k_hi, k_lo;              // windows per image in the high / low branch (the rest is pruned)
    int n_slots;                 // B*(k_hi+k_lo) windows that are computed
    int rows_hi, rows_lo;        // valid rows per region (B*k*49)
    int base_lo;                 // first row of the low region (multiple of REGION_ALIGN)
    int rows_total;              // multiple of REGION_ALIGN
    FastDiv by_nW, by_nWc, by_hi, by_lo;   // quotients by nW, nWc, k_hi and k_lo (1 where the count is 0)
};

// row -> branch, canonical slot-major row (g*49+t) and source pixel index (or -1)
struct RowInfo { int branch; int canon; int pix; int win; };

__device__ __forceinline__ RowInfo row_info(const Geom& G, const int* __restrict__ perm, int row)
{
    RowInfo ri;
    int r = row, k = G.k_hi, jbase = 0, valid_rows = G.rows_hi;
    ri.branch = 0;
    if (row >= G.base_lo) { r = row - G.base_lo; k = G.k_lo; jbase = G.k_hi; valid_rows = G.rows_lo; ri.branch = 1; }
    if (r >= valid_rows) { ri.canon = -1; ri.pix = -1; ri.win = -1; return ri; }
    int s = r / TOK, t = r - s * TOK;
    int b = ri.branch ? G.by_lo(s) : G.by_hi(s), j = jbase + (s - b * k);
    int w = perm[b * G.nW + j];
    int wr = G.by_nWc(w), wc = w - wr * G.nWc, tr = t / WS, tc = t - tr * WS;
    int pr = wr * WS + tr + G.shift; if (pr >= G.Hp) pr -= G.Hp;
    int pc = wc * WS + tc + G.shift; if (pc >= G.Wp) pc -= G.Wp;
    ri.canon = (b * G.nW + j) * TOK + t;
    ri.win = w;
    ri.pix = (pr < G.H && pc < G.W) ? (b * G.H + pr) * G.W + pc : -1;
    return ri;
}

}  // namespace mixaq
