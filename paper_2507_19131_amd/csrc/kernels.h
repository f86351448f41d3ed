// Argument blocks and launchers of the gfx950 kernels (host side sees only this).
#pragma once
#include "block_plan.h"
#include "mixaq_dev.h"
#include "product_plan.h"

namespace mixaq {

// Host side: the GELU_K x 4 coefficient table of gelu_pinned (api.hip uploads it once per block).
void gelu_table(float* tab);

struct LnArgs {
    const int* perm;                 // [B,nW] (gather only)
    const float* src;                // feature map (gather) or h rows [rows,C]
    const float* gamma[2];
    const float* beta[2];
    QDev q[2];
    float eps;
    int8_t* out;                     // operand fragments
    int* row_pix;                    // [rows] written by the gather, read otherwise
    int* row_canon;                  // [rows]
    int8_t* tap;                     // slot-major copy or NULL
};

struct GemmArgs {
    const int8_t* A;                 // activations, operand fragments (FC1, FC2: k in the order of the result registers)
    const v4i* Wp;                   // packed weights [N/32][K/32][64 lanes] x 16 bytes
    int K, N, nb_per_block;
    const float* m[2];               // s_in * s_w[n] per branch
    const float* bias[2];
    const int* negcorr[2];           // -zp_in * sum_k W[n,k]
    QDev q[2][3];                    // output quantizers (QKV: q,k,v; FC1: [0])
    int8_t* out8;                    // codes: [rows,N] (QKV), operand fragments of FC2 (FC1)
    float* outf;                     // [rows,N] (proj)
    const float* resid;              // [rows,N] (FC2)
    const float* x;                  // feature map, shortcut of the first residual (proj)
    float* y;                        // output map (FC2 scatter)
    const int* row_pix;
    const int* row_canon;
    int32_t* tap_acc;
    int8_t* tap_code;
    float* tap_f;
    const float4* gelu_tab;          // [GELU_K] cubic coefficients (FC1 epilogue)
    const GeluStep* steps[2];        // or, not NULL, the table of steps of each branch
    GeluIndex step_index[2];
    int step_pieces[2];
};

struct AttnArgs {
    const int8_t* qkv;               // [rows,3C]
    const int* perm;
    const float4* bias2;             // [4 mask types][heads][13 key quads][64 queries][4 keys], (bias+mask)*log2e
    float m2[2];                     // s_q*s_k/sqrt(d)*log2e
    float m_o[2];                    // s_p*s_v
    QDev qp[2], qo[2];
    int8_t* out;                     // operand fragments
    int32_t* tap_s;
    int8_t* tap_p;
    int32_t* tap_o;
    int8_t* tap_code;
    int floor[2];                    // which exponents need their floor: bit 0 windows without, bit 1 windows with masked pairs
};

struct WinArgs {                     // fused window kernel (gather + LN1 + QKV + attention)
    const float* x;
    const int* perm;                 // selection list, or ...
    const double* scores;            // ... the scores: every workgroup ranks its own window ([B,nW]; NULL = use perm)
    int* perm_out;                   // with scores: receives the selection list
    float* y;                        // with scores: pruned windows are forwarded here
    // per branch one block of 32-bit words, staged in LDS by every workgroup (the constants of its own heads only):
    // [LN1 gamma | LN1 beta] (C words each), then per head [q|k|v][m | bias | negcorr] (32 words each; negcorr integers)
    const float* params[2];
    float eps;
    QDev q_in[2];
    const v4i* Wqkv;                 // packed, natural k order
    QDev q_qkv[2][3];
    const float4* bias2;
    float m2[2], m_o[2];
    QDev qp[2], qo[2];
    int8_t* codes;                   // wide blocks: LN1 codes, operand fragments of 64 rows per slot (ln_window_kernel -> window_kernel)
    int8_t* out;                     // attention output codes
    int out_pack;                    // 0: int8 containers; 1, 2: the low region's rows packed (see packed_codes); PACK_FRAG: fragments
    int* row_pix;
    int* row_canon;
    int8_t* tap_a1; int32_t* tap_acc; int8_t* tap_qkv; int32_t* tap_s; int8_t* tap_p; int32_t* tap_o; int8_t* tap_code;
    int floor[2];                    // which exponents need their floor: bit 0 windows without, bit 1 windows with masked pairs
    bool taps;                       // any tap pointer set
    bool magic_sums;                 // negcorr words are SUM_MAGIC_BITS more (see sum_value)
};

struct TokArgs {                     // fused token kernel (proj + LN2 + FFN + scatter)
    const int8_t* ao;                // [rows,C]
    int ao_pack;                     // as WinArgs::out_pack
    const float* x;
    float* y;
    const int* row_pix;
    const int* row_canon;
    const v4i* Wproj;                // natural k order
    const v4i* W1;                   // k order of the MFMA result registers
    const v4i* W2;
    // per branch one block of 32-bit words, staged in LDS by every workgroup:
    // [proj m | proj bias | proj negcorr | LN2 gamma | LN2 beta | fc2 m | fc2 bias | fc2 negcorr] (C words each),
    // then [fc1 m | fc1 bias | fc1 negcorr] (4C words each); negcorr words are integers
    const float* params[2];
    float eps;
    QDev q_fc1in[2], q_fc2in[2];
    int32_t* tap_acc_proj; float* tap_h; int8_t* tap_a2; int32_t* tap_acc_fc1; int8_t* tap_g; int32_t* tap_acc_fc2; float* tap_y;
    const float4* gelu_tab;          // [GELU_K] cubic coefficients
    const GeluStep* steps[2];        // per branch the table of steps (see gelu_steps.h) and its 1 KB pieces ...
    GeluIndex step_index[2];
    int step_pieces[2];
    bool short_forms;                // ... used where both branches have one and the negcorr words of proj and fc1 are SUM_MAGIC_BITS more
    bool taps;
};

bool channels_supported(int C);
bool fused_token_supported(int C, int mlp_ratio);
// chains: how many launches like this one run beside each other (the two chains of a stage)
void launch_window(const Geom& G, const WinArgs& A, int chains, hipStream_t st);
void launch_token(const Geom& G, const TokArgs& A, int chains, hipStream_t st);
// both halves in one launch, where block_plan.h says so and the sums and the GELU take their short forms (one chain, no taps); false:
// nothing was launched
bool launch_block(const Geom& G, const WinArgs& W, const TokArgs& T, int chains, hipStream_t st);
bool launch_score(const Geom& G, const float* x, int mode, float eps, const float* gm, const float* bt, double* scores,
                  hipStream_t st);
void launch_select(const double* scores, int B, int nW, int reverse, int* perm, hipStream_t st);
void launch_bypass(const Geom& G, const int* perm, const float* x, float* y, hipStream_t st);
bool launch_ln_quant(const Geom& G, const LnArgs& A, bool gather, hipStream_t st);
void launch_gemm(const Geom& G, const GemmArgs& A, int epi, hipStream_t st);
void launch_attn(const Geom& G, const AttnArgs& A, hipStream_t st);

}  // namespace mixaq
