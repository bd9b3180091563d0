// Internal declarations shared by the translation units of librapid_hip.so (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "rapid.h"

namespace rapid {

typedef unsigned short bf16_t;  // raw bf16 bits in memory

static inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// Leading dimension (bf16 elements) for a row of x elements (x a multiple of 64): one extra
// 128-byte line when the row would otherwise span an even number of lines.  Consecutive rows of an
// operand tile are read for the same k at the same time; with an odd line stride they fall on
// different L2 / HBM channels instead of piling onto one or two.
static inline int64_t padded_ld(int64_t x) { return ((x / 64) % 2 == 0) ? x + 64 : x; }

// device counters written by the compaction step: [0] = M (valid tokens), [1] = M rounded up to 256
enum { CNT_M = 0, CNT_MR = 1, CNT_WORDS = 64 };

// One entry of the chunk table of the cached backward (int32 x CH_WORDS per chunk): words 0 and 1 are
// laid out like the counters above, so a kernel that is given `table + CH_WORDS * c` as its counters
// works on chunk c alone.  Chunk c owns the compact rows [c * Rcap, c * Rcap + rows).
enum { CH_M = 0,      // end of the chunk's valid rows (absolute compact row index)
       CH_MR = 1,     // that end rounded up to a row tile
       CH_G0 = 2,     // first generation of the chunk
       CH_G1 = 3,     // one past its last generation
       CH_ROWS = 4,   // valid rows
       CH_LIVE = 5,   // end of the rows that carry gradient (they come first; see IdleArgs); CH_LIVE, CH_LIVER lie
       CH_LIVER = 6,  // like CNT_M, CNT_MR: a kernel given tab + CH_LIVE as its counters stops at them
       CH_WORDS = 8 };

constexpr int ROW_TILE = 256;  // compact rows are padded to this
constexpr int K_TILE = 64;     // contraction tile of the MFMA kernels (bf16 elements)

// ---- reductions.hip ---------------------------------------------------------------------------
// IdleArgs (idle == NULL: off): generations whose coefficient is zero whatever their log-probs are (all rewards
// of the group exactly 0, or a coefficient override of 0) are marked in idle [N] and placed behind the others
// inside their chunk; the chunk's CH_LIVE / CH_LIVER say where the rows that carry gradient end.
struct IdleArgs {
    const float* rewards = nullptr;        // [N]
    const float* coef_override = nullptr;  // [N] or NULL; if given it alone decides
    int32_t* idle = nullptr;               // out [N]
    int32_t* len_live = nullptr;           // scratch [N]
    int32_t* cu_live = nullptr;            // scratch [N + 1]
    int32_t* live_group = nullptr;         // scratch [K]
};
// What the plan of a batch is made from and what it fills in (see plan_kernel).  cu [N + 1]: prefix sum of seq_len [N].
// tab NULL: one region; counts (optional) = M and M rounded up to a row tile.
// With tab the generations are dealt to at most Cmax chunks of at most Rcap compact rows
// each, whole groups (maximal runs of equal group id) at a time, in order, each chunk as full as it gets; chunk c's
// rows start at compact row c * Rcap.  Writes the chunk table `tab` [Cmax][CH_WORDS], gen_row0 [N]
// (compact row of each generation's first token, -1 for a generation that was left out),
// gen_chunk [N], and counts[CNT_M] = the tokens that were placed.
// Cmax == 1: one chunk takes every generation, groups may lie anywhere; tokens past Rcap are left
// out (RAPID_STATUS_TOKEN_BOUND).  Cmax > 1: a group whose members are not adjacent, or whose tokens
// exceed Rcap, sets RAPID_STATUS_GROUP_LAYOUT; more chunks than Cmax sets RAPID_STATUS_TOKEN_BOUND.
// runs [3K + 1] (optional): where each group lies in the batch; given to launch_group_advantage
// it lets a group that is one run of the batch look at that run alone.  lam_state (optional): set to -infinity.
struct PlanArgs {
    int64_t N = 0, K = 0;
    const int32_t* gid = nullptr;
    int32_t *seq_len = nullptr, *cu = nullptr, *counts = nullptr;
    int64_t Rcap = 0;     // with tab
    int32_t* tab = nullptr;
    int Cmax = 0;
    int32_t *gen_row0 = nullptr, *gen_chunk = nullptr, *runs = nullptr;
    double* lam_state = nullptr;
    IdleArgs idle;
    int32_t* dev_status = nullptr;
};
struct ZeroWords { int32_t* p[2] = {nullptr, nullptr}; int64_t n[2] = {0, 0}; };
void launch_plan(const uint8_t* mask, int64_t N, int64_t T, const PlanArgs& plan, hipStream_t st);
// The compact rows of a planned batch (rows.hip): what is not wanted is NULL.
struct RowsArgs {
    const uint8_t* mask = nullptr;
    int64_t N = 0, T = 0;
    // generation n's rows begin at first_row[n] (negative: left out), inside its region of `region` rows; limits[e * stride]:
    // counters of region e < entries.  first_row NULL: no plan was made; the rows are the valid positions in order, and their
    // number goes to counts_out
    const int32_t *first_row = nullptr, *limits = nullptr;
    int64_t region = 0;
    int stride = 0, entries = 0;
    int32_t* counts_out = nullptr;
    int32_t* row_index = nullptr;               // out: flat position of every row
    const int32_t* tokens = nullptr;            // [N, T]
    int64_t V = 0;
    int32_t *tokc = nullptr, *seqc = nullptr;   // out: token id and generation of every row
    int32_t* dev_status = nullptr;
    float *zero_a = nullptr, *zero_b = nullptr;   // [N, T]: zeros at the positions without a row
    uint32_t* dhidden = nullptr;                // [N, T] rows of words_per_row: zeros at masked positions and those of generations
    int64_t words_per_row = 0;                  // that idle [N] marks
    const int32_t* idle = nullptr;
    // packed hidden rows (bf16), zeros in columns d .. Cpad and in the rows that fill a region's last row tile up
    const bf16_t* hidden = nullptr;
    int64_t d = 0;
    bf16_t* Hc = nullptr;
    int64_t ldk = 0, Cpad = 0;
    const bf16_t* rms_weight = nullptr;         // normalised on the way; inv_rms: 1 / sqrt(mean(x^2) + eps) of every row
    float rms_eps = 0.f;
    float* inv_rms = nullptr;
    // logit of the sampled token (W: a token's weights in a row of ldw, or with `gather` in a column)
    const bf16_t* W = nullptr;
    int64_t ldw = 0;
    bool gather = false;
    float inv_temp = 1.f;
    float *zy = nullptr, *refz = nullptr;
    const float* ref_logp = nullptr;            // [N, T]
};
// Positions up to which the rows may do without a plan (first_row NULL): every wave then counts the batch's mask up to its place.
// Log-probs at d = 1024, V = 256 without a plan and with one: 64 x 32 positions 35 and 38 us, 64 x 64 42 and 45, 64 x 128 57 and 60;
// past the bound it depends on the shape (64 x 250 78 and 84, 1024 x 16 98 and 81).
constexpr int64_t ROWS_WITHOUT_PLAN = 8192;
// Positions per generation up to which calls with gradient rows take rows_by_position_kernel, whose waves count a generation's
// mask up to their place.  Steps of V = 256 by position and with an index of the rows, cached: 64 x 4095, d = 1024 961 and 975 us, 64 x 512
// 192 and 197, 1024 x 250 1022 and 974; just past the bound by position is still ahead (64 x 4097 947 and 963, 16 x 8192 551 and
// 555), but what a wave counts grows with the length.
constexpr int64_t BY_POSITION_T = 4096;
// rows: upper bound of the compact rows, padding included
void launch_compact_rows(const RowsArgs& a, int64_t rows, hipStream_t st);
void launch_rows(const RowsArgs& a, bool by_position, int64_t rows, hipStream_t st);   // its part in rows.hip
void launch_fill_f32(float* p, int64_t n, float v, hipStream_t st);
// lse/logp from per-slot partial (max, sumexp) and the gathered logit, compact rows [row0, row0 + rows_max);
// the partials of row j sit at column j - row0
void launch_merge_lse(const float* part_max, const float* part_sum, int P, int64_t ld_part,
                      const float* zy, const int32_t* row_index, const int32_t* counts, int64_t row0,
                      int64_t rows_max, float* lse_c, float* logp_out, float* lse_out, hipStream_t st);
// The estimator kernels take `gen_range` (device, two words: first generation and one past the last; NULL =
// all N): they then touch only those generations.
// tsum/tmax (NULL or [N]): per generation, sum and log-maximum of its tokens' (clipped if clip_tokens) ratios
void launch_seq_logratio(const float* logp_cur, const float* logp_behav, const uint8_t* mask, int64_t N,
                         int64_t T, float* tok_logratio_out, double* s64, float* s32, float eta, int clip_tokens,
                         double* tsum, double* tmax, const int32_t* gen_range, int32_t* dev_status, hipStream_t st);
// weights from s64 if given, else from s32, else 1; adv64 (NULL or [N]): the advantages before rounding to float.
// baseline_mode 0..2 as in rapid.h.
void launch_group_advantage(const float* rewards, const int32_t* group_ids, const float* s32, const double* s64,
                            int64_t N, int64_t K, float eta, int baseline_mode, float* adv, double* adv64,
                            float* weight, float* gmean, float* gstd, int32_t* gsize, const int32_t* gen_range,
                            int32_t* dev_status, hipStream_t st, const int32_t* runs = nullptr);
// Token-level clipped surrogate with KL penalty (the loss step of the GRPO / DAPO baselines).
// Advantage: (R - group mean) / (group std + adv_eps), the std with divisor N_k - std_ddof.
struct ClipArgs {
    const float* logp_cur; const float* logp_old; const float* logp_ref;   // [N,T]; old NULL: ratios 1; ref NULL: no KL term
    const int32_t* seq_len; const int32_t* counts;   // counts[CNT_M]: tokens of the call
    int64_t N, T, K;
    float eps_low, eps_high, kl_beta, loss_scale; int norm_mode;
    const float* rewards; const int32_t *group_ids, *runs; float adv_eps; int std_ddof;
    float* adv;                                      // [N]
    double* adv64;                                   // NULL, or [N] scratch: launch_clip_advantages forms the advantages
    // the generations' compact rows (as in RowsArgs), and dLoss/dlogp of the rows below row_counts[CNT_MR]
    const int32_t *first_row, *row_index, *row_counts; int64_t region;
    float* rowg;
    int32_t* dev_status;
};
// Generations up to which each one looks through its group (or through the whole batch where some group lies scattered); above, a
// launch does it per group, because all of them looking is quadratic work.  Steps (d = 16, V = 40) with each looking and with the launch:
// 2048 x 8 positions in groups of four 200 and 203 us, as one group 212 and 207; 4096 x 4 206 and 210, 237 and 222, scattered 223 and 220;
// 8192 x 2 219 and 224, 285 and 249, scattered 266 and 253; 20 000 x 1 302 and 310, 794 and 374.
constexpr int64_t CLIP_SCAN = 4096;
// with adv64, once a call and behind its plan
void launch_clip_advantages(const ClipArgs& a, hipStream_t st);
// advantages, the rows' coefficients, and per generation (in gen_range): its share of the loss, its clipped tokens, the sum of
// its tokens' KL estimates
void launch_clip_generations(const ClipArgs& a, const int32_t* gen_range, double* loss_n, double* clipped_n, double* kl_n, hipStream_t st);
// loss and diagnostics from the per-generation sums
void launch_clip_finish(const double* loss_n, const double* clipped_n, const double* kl_n, int64_t N, const int32_t* counts,
                        float* loss_out, rapid_clip_pg_diag* diag, hipStream_t st);
// tsum/tmax given: token-level outer weight (g_n is then the generation's factor without a ratio).
// Three uses.  Whole batch (gen_range, lam_state NULL): coefficients, scale lambda, loss, diagnostics.
// One chunk of the cached backward (gen_range and lam_state given): coefficients of the chunk's generations
// only, scaled by exp(-Lambda) with Lambda = max(lam_state[0], the chunk's own lambda) (0 if not normalized);
// writes Lambda back to lam_state[0] and to lam_chunk[0], and to beta_out[0] the factor
// exp(old Lambda - new Lambda) that the gradient sums accumulated so far have to be multiplied by; no loss,
// no diagnostics.  Closing pass (write_g = 0): loss and diagnostics of
// the whole batch, no coefficient is written.
struct CoefArgs {
    const double* s64; const float* adv; const double* adv64; const float* coef_override; int64_t N;
    float eta; int coef_mode; float loss_scale; int normalized;
    const double* tsum; const double* tmax; const int32_t* counts;
    float* g; double* g64; float* loss_out; rapid_iw_pg_diag* diag;
    const int32_t* gen_range; double* lam_state; double* lam_chunk; float* beta_out; int write_g;
};
void launch_coefficients(const CoefArgs& a, hipStream_t st);
// The estimator of a call that works on one chunk of rows from row 0 on, in one block for a batch that fits (see
// small_estimator_kernel): all of it, or what lies between the log ratios and the rows' coefficients.
// tok_lr may be NULL; of coef, what the caller hands in and the outputs count, and (not all of it) s64, tsum, tmax, g, g64.
struct EstimatorArgs {
    const float *logp_cur, *logp_behav;    // behav NULL: ratios 1
    const uint8_t* mask;
    int64_t N, T, K;
    const float* rewards;
    const int32_t* group_ids;
    int baseline_mode, clip_tokens, per_token;
    float *tok_lr, *s32, *adv;
    const int32_t *seqc, *row_index, *row_counts;
    float* rowg;
    int32_t* dev_status;
    CoefArgs coef;
};
enum { ESTIMATOR_LAUNCHES = 0, ESTIMATOR_GENERATIONS, ESTIMATOR_ONE };
int small_estimator_fits(int64_t N, int64_t T, int64_t K);
void launch_small_estimator(const EstimatorArgs& a, bool tokens, hipStream_t st);
// rowg[j] = dL/dlogp of compact row j in [row0, row0 + rows_max) (0 for padding rows): g of its generation,
// times its own ratio if per_token
void launch_row_coefficients(const float* g, const double* g64, const int32_t* seqc, const int32_t* row_index,
                             const int32_t* counts, const float* logp_cur, const float* logp_behav, int per_token,
                             float eta, int clip_tokens, int64_t row0, int64_t rows_max, float* rowg, hipStream_t st);
// cached backward with normalized gradients: every valid dhidden row of generation n is multiplied by
// exp(lam_chunk[gen_chunk[n]] - lam_state[0]) (the scale its chunk used against the final one)
void launch_rescale_rows(void* dhidden, const uint8_t* mask, int64_t N, int64_t T, int64_t d, const int32_t* gen_chunk,
                         const double* lam_chunk, const double* lam_state, hipStream_t st);
// dst[i] += src[i]
void launch_f32_add(const float* src, float* dst, int64_t n, hipStream_t st);
void launch_f32_to_bf16(const float* src, bf16_t* dst, int64_t n, hipStream_t st);

// ---- pack.hip ---------------------------------------------------------------------------------
// dst[r][c] (ld_dst) = src[r][c] for r < R, c < C else 0, over r < Rpad, c < Cpad.
void launch_copy_pad_bf16(const bf16_t* src, int64_t ld_src, bf16_t* dst, int64_t ld_dst, int64_t R, int64_t C, int64_t Rpad,
                          int64_t Cpad, hipStream_t st);
// dst = src [R, C] in zero-padded tile blocks of RB rows x 64 columns (see block_rows_bf16_kernel); the second one takes
// the transpose of src [R, C], so that the blocks run over src's columns.
void launch_block_rows_bf16(const bf16_t* src, int64_t ld, bf16_t* dst, int64_t R, int64_t C, int64_t Rpad, int64_t Cpad, int RB,
                            hipStream_t st);
void launch_transpose_blocks_bf16(const bf16_t* src, int64_t ld_src, bf16_t* dst, int64_t R, int64_t C, int64_t Rpad, int64_t Cpad,
                                  int RB, hipStream_t st);
// dst[c][r] (ld_dst) = src[r][c] for r < R, c < C else 0, over r < Rpad, c < Cpad.
void launch_transpose_pad_bf16(const bf16_t* src, int64_t ld_src, bf16_t* dst, int64_t ld_dst, int64_t R,
                               int64_t C, int64_t Rpad, int64_t Cpad, hipStream_t st);

// both packed copies of W in one pass: Wvd (rows up to Vpad, columns up to dpad) and the tile blocks of RB rows x 64 columns
void launch_pack_both_bf16(const bf16_t* W, bool vd, int64_t d, int64_t V, bf16_t* Wvd, int64_t ldk, int64_t dpad, bf16_t* blocks,
                           int64_t dpadR, int RB, int64_t Vpad, hipStream_t st);

// ---- rmsnorm.hip ------------------------------------------------------------------------------
// dh [N*T, d] holds dL/dh at the valid positions of the compact rows, which come in regions of region_rows rows with their
// counters at counts[g * stride]; it becomes dL/dx in place, and dweight [d] (may be NULL) dL/dweight.  part: scratch of part_bytes
// (128 MiB) for the partial sums; part_512: scratch that has room for a row of d sums per 512 rows of every region.
void launch_rmsnorm_backward(const bf16_t* x, bf16_t* dh, int64_t d, const bf16_t* weight, const int32_t* row_index,
                             const int32_t* counts, int stride, int regions, int64_t region_rows, const float* inv_rms, float* part,
                             size_t part_bytes, float* part_512, float* dweight, hipStream_t st);

// ---- gemm_bf16.hip ----------------------------------------------------------------------------
// The head as the caller has it.  mode says how a kernel reads it: from a packed copy (the argument structs hold those),
// or in place, stored [V, d] or [d, V].
enum { W_PACKED = 0, W_VD = 1, W_DV = 2 };
struct WInPlace {
    const bf16_t* W = nullptr;
    int64_t d = 0, V = 0;
    int mode = W_PACKED;
};

struct FwdArgs {          // logits tile -> per-slot (max, sumexp) and gathered logit
    WInPlace w;
    const bf16_t* Wvd;    // [Vpad, dpad] (packed)
    const bf16_t* Hc;     // [Mmax_pad, dpad]
    int64_t dpad;         // contraction extent (multiple of 64)
    int64_t ldk;          // leading dimension of Wvd and Hc (elements)
    int tilesV, tilesM;   // 256-tiles (tilesM: row tiles of this launch, from row0 on; rows past the last token are skipped)
    int64_t row0;         // first compact token row of this launch
    int64_t V;
    float inv_temp;
    const int32_t* counts;
    float* part_max;      // [P][ld_part], P = tilesV * 2
    float* part_sum;
    int64_t ld_part;
    int gi;               // tiles along i that share one j before the order moves on (L2 blocking)
    bf16_t* zc;           // NULL, or [rows, ldz]: the kernel also stores exp(logit - refz[row]) there; refz must be set
    int64_t ldz;
    const float* refz;    // [Mmax_pad] reference of the stored exponentials
    int32_t* dev_status;  // may be NULL
    int64_t part_row0 = 0;   // compact row whose partials sit in column 0 of part_max / part_sum
    int64_t zc_row0 = 0;     // compact row stored in row 0 of zc
    const bf16_t* WvdB = nullptr;   // if set: W blocked per (256-row tile, K step of 32) (launch_block_w32); selects the
                                    // kernel that runs two workgroups per CU
    int k32_mode = 1;               // with WvdB: 1 = two 4-wave workgroups per CU on 256 x 128 tiles, 2 = one 8-wave
                                    // workgroup per CU on 256 x 256 tiles with requests three K steps ahead
};
void launch_fwd_lse(const FwdArgs& a, hipStream_t st);
// out [Vpad * dpad]: Wvd [Vpad, ldk] in blocks of 256 rows x 32 columns, in the LDS order of the two-workgroup forward
void launch_block_w32(const bf16_t* Wvd, int64_t ldk, bf16_t* out, int64_t Vpad, int64_t dpad, hipStream_t st);
int fwd_slots_per_tile();

struct DzArgs {           // logits tile -> dz = g (onehot - p) / temperature, bf16 [Mc, Vpad]
    WInPlace w;
    const bf16_t* Wvd;
    const bf16_t* Hc;     // already offset to the chunk's first row
    int64_t dpad, ldk;
    int tilesV, tilesM;   // tilesM = chunk rows / 256
    int64_t V, Vpad;
    int64_t ldz;          // leading dimension of dz
    float inv_temp;
    int64_t m0;           // first compact row of the chunk
    const int32_t* tokc;  // full arrays (indexed by compact row)
    const float* lse_c;
    const float* rowg;    // dL/dlogp per compact row
    const int32_t* counts;
    bf16_t* dz;           // [Mc, Vpad]
    int gi;               // tiles along i that share one j before the order moves on (L2 blocking)
};
void launch_dz(const DzArgs& a, hipStream_t st);
// turns the ratios a storing forward left in u [rows_max, ldz] (row 0 = compact row row0) into the
// backward's operands: the sampled token's element of each row, the row factors rowc, and Hc scaled by
// them in place (Hc, tokc, zy, refz, lse_c, rowg, rowc are indexed by compact row)
void launch_cache_finish(bf16_t* u, int64_t ldz, bf16_t* Hc, int64_t ldk, const int32_t* tokc,
                         const float* zy, const float* refz, const float* lse_c, const float* rowg, float inv_temp,
                         const int32_t* counts, int64_t row0, int64_t rows_max, float* rowc, int32_t* dev_status,
                         hipStream_t st);

struct DhArgs {           // dH[row, :] = dz[row, :] . Wdv^T
    WInPlace w;
    const bf16_t* Wdv;    // [dpadR, Vpad] (packed)
    const bf16_t* WdvB;   // the same, tile-blocked (blocks of tile-rows x 64 columns), or NULL
    const bf16_t* dz;     // [Mc, Vpad]
    int64_t Vpad;         // contraction extent
    int64_t ldv;          // leading dimension of Wdv and dz
    int64_t d, dpadR;     // dpadR: d rounded up to tiles of dtile (256, 224, 192 or 128)
    int dtile;
    int tilesM;
    int64_t m0;
    const int32_t* row_index;
    const int32_t* counts;
    const float* rowc;    // NULL, or one factor per compact row applied to the result
    unsigned* pace;       // NULL, or one word, zero at launch: arrival counter of the launch's workgroups
    int pace_every;       // K steps between meetings (power of two)
    bf16_t* dhidden;      // [N*T, d]
    int gi;               // tiles along i that share one j before the order moves on (L2 blocking)
    float* part = nullptr;    // NULL, or scratch of part_bytes (128 MiB): lets the kernel cut a partly filled last round of
    size_t part_bytes = 0;    // tiles along the contraction
};
void launch_dh(const DhArgs& a, hipStream_t st);
bool short_dh_packed(int64_t d, int64_t tilesM, int64_t V);   // whether dHidden wants tiles of 128 x 128 from a packed copy
size_t dh_part_bytes();   // scratch that lets a dHidden or dW launch cut its last round

struct DwArgs {           // dW (+)= Hc^T . dz over the chunk's rows
    const bf16_t* dz;     // [Mc, Vpad] chunk (rows = tokens)
    const bf16_t* Hc;     // [Mmax_pad, >= dpadR; + 64 with tiles of 192], already offset to the chunk's first row
    int64_t Mc;           // rows of the chunk buffer (contraction extent is min(Mc, rows left))
    int64_t ldz, ldH;     // leading dimensions of dz and Hc
    int64_t d, dpadR, V, Vpad;
    int dtile;            // 256, 192 or 128
    int64_t m0;
    const int32_t* counts;
    float* dW;            // fp32, layout per w_layout
    bf16_t* dW16 = nullptr;   // if set the result goes here, rounded once (the old value of beta = 1 still comes from dW)
    int w_layout;
    int beta;             // 0 overwrite, 1 accumulate
    const float* beta_scale = nullptr;   // NULL, or device: with beta = 1 the old value is multiplied by beta_scale[0] first
    int gi;               // vocabulary tiles that share one tile of d before the order moves on (L2 blocking)
    float* part = nullptr;    // as in DhArgs
    size_t part_bytes = 0;
};
void launch_dw(const DwArgs& a, hipStream_t st);
// whether the batch is small enough for both, of the same rows, to run side by side in one launch, and that launch
bool dh_dw_together(const DhArgs& h, const DwArgs& w);
void launch_dh_dw(const DhArgs& h, const DwArgs& w, hipStream_t st);
void set_waves_per_workgroup(int n);   // 4, 8 or 16 waves per contraction workgroup
bool default_waves();                  // each kernel runs its own choice
void set_dw_deep(int on);              // dW with K steps of 32 rows and requests three steps ahead
void set_cu_count(int n);              // compute units of the device: the contraction kernels launch one workgroup each


void launch_sgd_step(float* master, const float* grad, int64_t n, float lr, void* w_out, int dtype, hipStream_t st);
void launch_adamw_step(float* master, const float* grad, float* m, float* v, int64_t n, float lr, float beta1, float beta2,
                       float eps, float weight_decay, int64_t step, void* w_out, int dtype, hipStream_t st);

// ---- probe.hip -----------------------------------------------------------------------------------
int run_mfma_probe(int random_operands, int iters, int num_cu, double* tflops_out, double* ms_out, hipStream_t st);

// ---- f32_path.hip -----------------------------------------------------------------------------
// C[i][j] (+)= alpha sum_k A(i,k) B(k,j), arbitrary strides, optional index maps, and a device-side
// row count.  Accumulates in fp64.
struct F32Gemm {
    const float* A; int64_t sa_i, sa_k;
    const int32_t* a_imap;   // optional: A row of i is a_imap[i0 + i]
    const int32_t* a_kmap;   // optional: A position of k is a_kmap[i0 + k]
    const float* B; int64_t sb_k, sb_j;
    float* C; int64_t sc_i, sc_j;
    const int32_t* c_rows;   // optional: C row of i is c_rows[i0 + i]
    int64_t I, J, Kd;
    int beta;
    const int32_t* counts; int64_t i0;   // if counts: I (or Kd when limit_k) is clipped to M - i0
    int limit_k;
    float alpha;
    int may_split;           // 1: the order of summation may depend on the shape (never for logits: two calls on one batch
                             // have to agree in every bit)
    int skip_last;           // 1: nothing to do if no row lies past this chunk (its C is still what this launch would form)
};
void launch_f32_gemm(const F32Gemm& g, hipStream_t st);
// dHidden (no maps on its contraction index) and dW (with one) of the same rows, in one launch if both are small
void launch_f32_gemm_pair(const F32Gemm& dh, const F32Gemm& dw, hipStream_t st);
// row-wise: lse, logp, gathered logit from a materialised logits chunk z [rows, V]
void launch_f32_row_lse(const float* z, int64_t V, int64_t rows, int64_t m0, const int32_t* tokc,
                        const int32_t* row_index, const int32_t* counts, float* lse_c, float* logp_out,
                        float* lse_out, hipStream_t st);
// in place: z -> dz = g (onehot - softmax) * inv_temp
void launch_f32_dz(float* z, int64_t V, int64_t rows, int64_t m0, const int32_t* tokc,
                   const float* lse_c, const float* rowg, float inv_temp, const int32_t* counts, hipStream_t st);

void set_error(const char* fmt, ...);

}  // namespace rapid
