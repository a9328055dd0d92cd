/*
 * psd.h -- C ABI of the keyed Poisson-race multi-draft speculative sampler on
 * MI355X (gfx950): drafting, verification and watermark detection from
 * "Watermarkable Multi-Draft Speculative Sampling via Poisson Processes".
 *
 * Conventions shared by every entry point
 * ---------------------------------------
 *  - Ownership: every pointer is owned by the caller.  The library never
 *    allocates or frees caller-visible memory and keeps no pointer after it
 *    returns.  Pointers marked "device" must point to device memory of the
 *    current HIP device; host pointers are marked "host".
 *  - Asynchrony: each call validates its arguments on the host, enqueues its
 *    kernels on `stream` and returns.  Outputs are valid once the stream has
 *    reached that point; the library never synchronises.  One call also uses
 *    a stream of its own (psd_verify, see there): its work there is ordered
 *    after the caller's earlier work on `stream` and before the caller's later
 *    work, through events.
 *  - Errors: any invalid scalar or missing required pointer returns PSD_E_ARG
 *    before anything is enqueued.  A failed launch returns PSD_E_HIP.  A
 *    workspace that is too small returns PSD_E_WORKSPACE.  The message of the
 *    last non-OK status of the calling thread is psd_last_error().  No C++
 *    exception crosses the ABI.
 *  - Logits: row-major with the vocabulary contiguous, float32 or bfloat16
 *    (psd_params.dtype).  A -inf logit means probability 0: that token is never
 *    selected.  A row without any finite logit yields token -1 and LSE -inf.
 *    NaN logits are a caller error (results undefined).
 *  - Temperatures are applied inside the kernels (logit / T).
 *
 * The keyed source (the paper's Pi(c) = G(k, Lambda(c)); Sec. 4.3, Sec. 5 and
 * the appendix "Algorithm Implementation"): the context of the token generated
 * at absolute 0-based position t is labelled by (key, t, last m tokens), folded
 * into a 64-bit Philox key kappa with Philox4x32-10 (Salmon et al., SC'11).
 * Clocks E_j[v] (slot j = list index, token v) are iid Exp(1) given kappa,
 * generated by one of two layouts (psd_clocks); both give the same law.
 *
 * The race (eq. EFR and the PFR-to-EFR reduction; non-identical proposals,
 * Prop. "heterogeneous PML bound"): draft k takes argmin_v ln E_k[v] - l_v/T_Q;
 * the target takes argmin over (v, j < K) of ln E_j[v] - l_v/T_P.  Exact ties go
 * to the lowest v, then the lowest j.
 */
#ifndef PSD_H
#define PSD_H

#include <stddef.h>
#include <stdint.h>

#include <hip/hip_runtime_api.h>

#ifdef __cplusplus
extern "C" {
#endif

#define PSD_ABI_VERSION 4
#define PSD_MAX_VOCAB (1 << 19) /* V <= 524288 */
#define PSD_MAX_DRAFTS 32       /* K */
#define PSD_MAX_GAMMA 32        /* gamma */
#define PSD_MAX_WINDOW 16       /* m */
#define PSD_MAX_BATCH (1 << 19) /* B */
#define PSD_MAX_TOP_K 256       /* top_k */

typedef enum {
    PSD_OK = 0,
    PSD_E_ARG = -1,         /* invalid argument, nothing enqueued */
    PSD_E_UNSUPPORTED = -2, /* valid but not implemented (reserved) */
    PSD_E_HIP = -3,         /* HIP runtime / launch failure */
    PSD_E_WORKSPACE = -4    /* workspace missing or too small */
} psd_status;

typedef enum { PSD_F32 = 0, PSD_BF16 = 1 } psd_dtype;

/* HET: K distinct drafters, draft k races slot k, the target races all K slots
 *      (augmented space V x [K], Prop. "heterogeneous PML bound").
 * MPFR: K identical drafters (Sec. 5, eq. MPFR; Alg. "Multi-Draft ... (Formal)";
 *      the direct finite-support sampler of the appendix on finite-support MPFR).
 *      The K paths hold the context tree: at depth s the paths with equal drafts
 *      at depths < s share one context c with multiplicity nu(c) = their count;
 *      c's proposal row is its lowest path's draft row (the others are read only
 *      for their LSE), and c's nu(c) drafts are the labels of the nu(c) smallest
 *      ln(E_0[v] + ... + E_j[v]) - l_v/T_Q over (v, j < nu(c)) under c's keyed
 *      source, the i-th smallest going to c's i-th path (increasing index).
 *      Target rows race slot 0 alone (MPFR(P, Pi(c), 1)); the walk is unchanged;
 *      detection scores the slot-0 clock (K = 1).  Drafting runs before the walk:
 *      the draft rows are streamed, and the contexts sampled by one launch per depth,
 *      or, when the block's (sequence, path) workgroups fit the device together, by one
 *      launch for every depth (each depth's contexts formed as the earlier drafts
 *      land; it may run beside the streaming launch, and reads a row itself that does
 *      not come in time); with a shared target chain, psd_verify races the chain beside
 *      it (see there). */
typedef enum { PSD_MODE_HET = 0, PSD_MODE_MPFR = 1 } psd_mode;

/* TREE: clocks of a slot built top-down over a fixed token hierarchy (8-token
 *       chunks, then 16-ary nodes of 128, 2048, 32768 tokens, root = all V):
 *       a node's minimum is Exp(1)/n at a uniform position; a node that does
 *       not hold its parent's minimum has minimum m_parent + E'/n; a token that
 *       is not its chunk's minimum has clock m_chunk + E'.  The race only
 *       expands nodes whose lower bound ln m - max(l)/T can still win.
 *       Node (level L, index i) draws Philox(ctr=(i, j, L, 2), kappa);
 *       token v draws word v&3 of Philox(ctr=(v>>3, j, 8+((v>>2)&1), 2), kappa).
 * FLAT: E_j[v] = -ln U(Philox(ctr=(v>>2, j, 0, 0), kappa)[v&3]).
 * U(w) = (2*(w>>9)+1) * 2^-24 in both layouts. */
typedef enum { PSD_CLOCKS_TREE = 0, PSD_CLOCKS_FLAT = 1 } psd_clocks;

typedef struct {
    uint64_t key;       /* watermark secret key */
    int32_t vocab;      /* V, 1 <= V <= PSD_MAX_VOCAB */
    int32_t num_drafts; /* K, 1..PSD_MAX_DRAFTS */
    int32_t ctx_window; /* m, 0..PSD_MAX_WINDOW: previous tokens hashed into the context label */
    float temp_target;  /* T_P > 0, finite */
    float temp_draft;   /* T_Q > 0, finite */
    int32_t dtype;      /* psd_dtype of every logits buffer */
    int32_t mode;       /* psd_mode */
    int32_t clocks;     /* psd_clocks */
    int32_t top_k;      /* 0: no truncation; 1..PSD_MAX_TOP_K: every row races only its top_k largest
                           logits (ties to the lowest token index) */
    float top_p;        /* 1: no truncation; (0, 1): then only the shortest prefix of those (logit
                           descending) whose probability at the row's temperature reaches top_p;
                           needs top_k >= 1.  Truncation (the paper's experiments: temperature,
                           top-k, top-p before the race) runs its own kernels: a selection per row
                           and one workgroup per sequence racing the kept lists with exact clocks;
                           LSE outputs are those of the kept sets. */
} psd_params;

typedef struct {
    int32_t batch;                /* B sequences, 1..PSD_MAX_BATCH */
    int32_t gamma;                /* draft length, 1..PSD_MAX_GAMMA */
    const int32_t *prefix_tokens; /* device [B][m]: the m tokens before start_pos, oldest first; -1 pads a
                                     text shorter than m.  May be NULL when m == 0. */
    const int64_t *start_pos;     /* device [B]: absolute 0-based position of the block's first token */
    void *workspace;              /* device scratch of workspace_bytes >= psd_workspace_bytes(), 256-byte
                                     aligned, owned by the caller; zero-filled before its first use
                                     (psd_workspace_clear).  Every value a call publishes in it is tagged
                                     with that call's 32-bit epoch, and the call's last workgroup resets
                                     the work queues and advances the epoch, so nothing needs clearing
                                     between calls, even of different shapes.  Clear it again after
                                     4294443007 calls, after a launch that did not run to completion, or
                                     to reset the error bits.  One call at a time per workspace. */
    size_t workspace_bytes;
    uint32_t *status;             /* device, nullable: one word that the call's last workgroup sets to the
                                     error bits of this call (0 = healthy; bits as in
                                     psd_workspace_errors), in stream order, without a host
                                     synchronisation.  With a bit set the call's outputs are unreliable. */
} psd_block;

/* Bytes of workspace for blocks of `batch` sequences and draft length `gamma`
 * under `params` (covers psd_draft and both target_rows modes of psd_verify; with
 * top_k > 0 it includes the kept lists of every row, 8 bytes per kept token).
 * Returns 0 for invalid arguments. */
size_t psd_workspace_bytes(const psd_params *params, int32_t batch, int32_t gamma);

/* Zero the whole workspace with a fill kernel on `stream` (work counter, epoch,
 * error bits and every slot).  Needed once after allocation; see psd_block. */
psd_status psd_workspace_clear(void *workspace, size_t workspace_bytes, hipStream_t stream);

/* Error bits recorded by kernels in the workspace since the last clear (sticky;
 * host pointer out; synchronises `stream`): bit 0 = a wait for another
 * workgroup's value hit its spin limit, bit 1 = a race's candidate list
 * overflowed.  0 = healthy; with a bit set the outputs of the calls since the
 * last clear are unreliable.  Each call's own bits also reach psd_block.status.
 *
 * The fused kernel is persistent: its grid is sized so that all its workgroups
 * are resident together, and a finishing workgroup waits (bounded) for values
 * that other workgroups publish.  If another kernel holds part of the device
 * at the same time, a wait can run out before its producer is scheduled: the
 * call then completes with bit 0 set rather than deadlocking. */
psd_status psd_workspace_errors(const void *workspace, hipStream_t stream, uint32_t *out_bits);

/* Draft depths [s_begin, s_begin + s_count) of every path (Sec. 4.3 and Sec. 5:
 * draft k at depth s races slot k of the source keyed by its own context
 * prefix || x^(k)_{<s}).
 *   draft_logits  device [B][K][s_count][V] (dtype), row (b,k,i) is depth s_begin+i
 *   draft_tokens  device [B][K][gamma] int32, in/out: depths < s_begin are read
 *                 (context), depths in the range are written
 *   draft_lse     device [B][K][gamma] float, nullable: ln sum_v exp(l_v/T_Q)
 * 0 <= s_begin, 1 <= s_count, s_begin + s_count <= gamma. */
psd_status psd_draft(const psd_params *params, const psd_block *block, int32_t s_begin, int32_t s_count,
                     const void *draft_logits, int32_t *draft_tokens, float *draft_lse, hipStream_t stream);

/* Verify one speculative block (Alg. "Multi-Draft ... (Formal)" with the
 * augmented-space coupling for K distinct drafters).
 *   target_rows   1: target_logits device [B][gamma+1][V]; depth s of the target
 *                    chain is raced in the context prefix || y_{<s} (the chain
 *                    never reads the drafts: stopping-time drafter invariance).
 *                 K: target_logits device [B][K][gamma+1][V]; row (b,k,s) is raced
 *                    in path k's context prefix || x^(k)_{<s}; the walk reads the
 *                    row of the lowest-index active path.
 *   draft_logits  device [B][K][gamma][V] or NULL.  Non-NULL: the drafts are
 *                 computed in the same fused kernel and written to draft_tokens;
 *                 NULL: draft_tokens [B][K][gamma] is an input.
 *   out_tokens    device [B][gamma+1] int32: emitted tokens, -1 past out_len
 *   out_len       device [B] int32: tau = tokens emitted (accepted + 1), 1..gamma+1
 *   target_lse    device [B][gamma+1] (or [B][K][gamma+1]) float, nullable
 *   draft_lse     device [B][K][gamma] float, nullable (only with draft_logits)
 *   target_tokens device [B][gamma+1] (or [B][K][gamma+1]) int32, nullable: every
 *                 target race winner, including depths past out_len
 * Walk: with A_0 = all paths, for s < gamma emit y_s; stop after it when y_s is
 * -1 or not a draft of an active path at depth s; else keep the active paths
 * that drafted y_s.  After gamma acceptances emit the bonus y_gamma.
 * Identical drafters (PSD_MODE_MPFR) with draft_logits and target_rows 1: the
 * target chain is raced, and the draft rows are streamed or sampled, on two library
 * streams of the current device (created at the first such call and kept until the
 * process ends) beside the launches on `stream`; `stream` waits for both through
 * events before the walk.
 * Under stream capture the whole call stays on `stream`.  Such calls on one
 * device share those streams (calls from several host threads are serialised
 * while they enqueue). */
psd_status psd_verify(const psd_params *params, const psd_block *block, int32_t target_rows,
                      const void *target_logits, const void *draft_logits, int32_t *draft_tokens,
                      int32_t *out_tokens, int32_t *out_len, float *target_lse, float *draft_lse,
                      int32_t *target_tokens, hipStream_t stream);

/* psd_verify without a caller workspace, for callers that cannot allocate device
 * memory (code being captured into a HIP graph, tight serving loops, harnesses
 * that forbid allocation).  Same arguments, results and asynchrony as
 * psd_verify, except that block->workspace must be NULL and
 * block->workspace_bytes 0: the call uses a fixed scratch array of 32 MiB per
 * device, defined in the library and held until the process ends.  A shape whose
 * workspace (psd_workspace_bytes) exceeds 32 MiB returns PSD_E_WORKSPACE (the
 * V=128256, K=4, gamma=4, B=64 block needs 19.98 MB).  The call allocates
 * nothing: its first call on a device looks up the array's address and zeroes it
 * with a fill kernel on `stream`.  Every call on a device shares that device's
 * array: calls that overlap on one device (other streams, other threads) race
 * and give wrong results; serialise them.  Error bits reach block->status. */
psd_status psd_verify_static(const psd_params *params, const psd_block *block, int32_t target_rows,
                             const void *target_logits, const void *draft_logits, int32_t *draft_tokens,
                             int32_t *out_tokens, int32_t *out_len, float *target_lse, float *draft_lse,
                             int32_t *target_tokens, hipStream_t stream);

/* Watermark detection (eq. S_A; Alg. "Compute Aaronson score ..."): for each
 * sequence i and position t in [n0[i], seq_len) with 0 <= tokens[i][t] < V,
 * A_t = -ln(1 - r_t), r_t = exp(-K min_{j<K} E_j[w_t]) in the context
 * (key, t, tokens[i][t-m..t-1]) (-1 before position 0).  Tokens outside [0, V)
 * are not scored.
 *   tokens        device [n_seq][seq_len] int32
 *   n0            device [n_seq] int32, first scored position (0 <= n0)
 *   out_score     device [n_seq] double: S_A = sum of A_t
 *   out_count     device [n_seq] int32: M = number of scored tokens
 *   out_per_token device [n_seq][seq_len] float, nullable: A_t, NaN where not scored */
psd_status psd_detect(const psd_params *params, int32_t n_seq, int32_t seq_len, const int32_t *tokens,
                      const int32_t *n0, double *out_score, int32_t *out_count, float *out_per_token,
                      hipStream_t stream);

/* Gamma-tail p-value of detection scores (App. "Gumbel Watermark": under the null
 * the M scored A_t are iid Exp(1), so S_A ~ Gamma(M, 1),
 * p_A = Gamma(M, S_A) / Gamma(M) and ANLPPT_A = -(1/M) ln p_A).  Computed in
 * double precision on the device, one wavefront per sequence, from the outputs of
 * psd_detect (or any caller's S_A and M).
 *   score        device [n_seq] double: S_A
 *   count        device [n_seq] int32: M
 *   out_log_p    device [n_seq] double: ln p_A (0 when M = 0 or S_A <= 0; NaN when
 *                M < 0 or S_A is NaN, or if the evaluation did not converge)
 *   out_anlppt   device [n_seq] double, nullable: ANLPPT_A (NaN when M <= 0)
 * Arguments are checked before anything is enqueued (PSD_E_ARG for n_seq < 0 or a
 * NULL required pointer with n_seq > 0); the caller owns every buffer. */
psd_status psd_detect_pvalue(int32_t n_seq, const double *score, const int32_t *count, double *out_log_p,
                             double *out_anlppt, hipStream_t stream);

/* Parameters of the further detection scores.  The paper fixes neither; the
 * library claims no default. */
typedef struct {
    double li_delta; /* Delta of Li et al.'s score h*_{gum,Delta}, 0 < Delta < 1 */
    double pl_eps;   /* eps of Lattimore's truncated power-law score, 0 < eps <= 1 */
} psd_score_params;

/* Four detection statistics of each sequence from the same pivots (App. "Gumbel
 * Watermark" and the appendices on Li et al.'s and Lattimore's scores): with the
 * target's clock c_t = K min_j E_j[w_t] (K = 1 in MPFR mode) and pivot r_t = e^{-c_t},
 * uniform under the null,
 *   S_A  = sum -log(1 - r_t)                                  (Aaronson)
 *   S_U  = sum r_t                                            (U-score)
 *   S_Li = sum log(k r_t^{Delta/(1-Delta)} + [q>0] r_t^{(1-q)/q}),
 *          k = floor(1/(1-Delta)), q = 1 - k (1-Delta)           (Li et al.)
 *   S_PL = sum min(eps^{-1/2}, (1-r_t)^{-1/2}) - (2 - sqrt(eps)) (Lattimore)
 * over positions t in [n0[i], seq_len) of row i with 0 <= tokens < V, in fp64.
 *   tokens      device, row i at tokens + i * row_stride (row_stride >= seq_len: a
 *               prefix of each row can be scored, e.g. for a detection token budget)
 *   out_scores  device [n_seq][4]: S_A, S_U, S_Li, S_PL;  out_count device [n_seq]: M
 * PSD_E_ARG for Delta outside (0, 1), eps outside (0, 1] or bad sizes/pointers. */
psd_status psd_detect_scores(const psd_params *params, const psd_score_params *score_params, int32_t n_seq,
                             int32_t seq_len, int32_t row_stride, const int32_t *tokens, const int32_t *n0,
                             double *out_scores, int32_t *out_count, hipStream_t stream);

/* Null-tail p-values of the four statistics (device [n_seq][4] in, [n_seq][4] out):
 * column 0 ln p_A exactly (the Gamma(M, 1) tail, as psd_detect_pvalue); columns 1-3
 * Chernoff bounds ln p <= min_{lam >= 0} M ln E[e^{lam h(U)}] - lam S over the null pivot
 * U ~ Unif(0, 1) -- the U-score's as the paper gives it (E[e^{lam U}] = (e^lam - 1)/lam),
 * the same construction for Li et al.'s and Lattimore's scores (their null MGFs by
 * quadrature).  0 when S is at most the null mean M E[h] or M = 0; NaN for M < 0 or a
 * NaN score.  ANLPPT = -ln p / M. */
psd_status psd_detect_scores_pvalue(const psd_score_params *score_params, int32_t n_seq, const double *scores,
                                    const int32_t *count, double *out_log_p, hipStream_t stream);

/* Detections at level alpha (Sec. 6 / App. "Drafter-substitution ablation": declare
 * detection when the null p-value is at most alpha; TPR@1%FPR is this count over
 * watermarked texts at alpha = 0.01, the empirical FPR the same over unwatermarked
 * ones): *out_count (device int32) = #{i < n : log_p[i * stride] <= ln alpha}. */
psd_status psd_detection_rate(int32_t n, const double *log_p, int32_t stride, double alpha, int32_t *out_count,
                              hipStream_t stream);

/* ---- multi-block generation ------------------------------------------------- */

/* Commit one verified block into the sequences' texts and set up the next block:
 * generation repeats blocks, each emitted token extends its sequence's text, and
 * the next block starts at the new length with the new context window (the
 * generation loop of Alg. "Batched-target direct-top-k MPFR speculative sampling"
 * and of App. F's formal multi-draft algorithm).  Asynchronous on `stream`.
 *   out_tokens, out_len  device [B][gamma+1], [B] int32 from psd_verify; out_len NULL
 *                 sets up the first block instead: length = m (the prompt)
 *   text          device [B][text_stride] int32, in/out: [0, m) holds the prompt and
 *                 [m, max_len) receives the emitted tokens (the tokens of a block past
 *                 max_len are dropped); a -1 token (a row with no finite logit) ends its
 *                 sequence and fills the rest of its text with -1
 *   length        device [B] int64, in/out: tokens in each text, m <= length <= max_len
 *   prefix_tokens device [B][m] int32, out: text[start - m, start) of the next block
 *   start_pos     device [B] int64, out: min(length, max_len - 1) -- a finished
 *                 sequence repeats its last block, whose tokens are not committed
 *   n_active      device int32, out: sequences with length < max_len
 * m = params->ctx_window; m < max_len <= text_stride. */
psd_status psd_advance(const psd_params *params, int32_t batch, int32_t gamma, int64_t max_len,
                       const int32_t *out_tokens, const int32_t *out_len, int32_t *text, int64_t text_stride,
                       int64_t *length, int32_t *prefix_tokens, int64_t *start_pos, int32_t *n_active,
                       hipStream_t stream);

/* A synthetic position-indexed language model, to drive and measure the loop with
 * no model: the target row of sequence b at absolute position t is a fixed function
 * of (seed, b, t), and drafter k adds noise keyed by (draft_seed, b, k, t), so the
 * generated text must equal plain keyed decoding with the target rows whatever the
 * drafts (App. C).  Definition, every fp32 operation rounded once (no fused
 * multiply-add), bf16 rows the round-to-nearest-even of the fp32 values; sm =
 * SplitMix64, lowbias32 = Wellons' 32-bit integer hash:
 *   R_T = sm(seed ^ sm(b << 32 | t)), R_P = sm(R_T ^ 0xD1B54A32D192ED03),
 *   R_D = sm(draft_seed ^ sm((k + 1) << 56 ^ b << 32 ^ t))   (t taken mod 2^32)
 *   rank r(v) = (a v + c) mod V: c = R_P mod V, a = (R_P >> 32) mod V (0 -> 1), moved
 *     up (wrapping V -> 1) to the first value coprime to V
 *   x = lo32(R) + v * 0x9E3779B9 (mod 2^32); a 32-bit word h gives two uniforms
 *     (lo16(h) + 1/2) / 2^16 and (hi16(h) + 1/2) / 2^16
 *   target n = (sum of the 4 uniforms of lowbias32(x), lowbias32(x ^ hi32(R_T)) - 2) * sqrt(3)
 *     with x from R_T; q(r) = fp32(bits(fp32(1 + r)) - 0x3F800000);
 *     w = fp32(-alpha * ln 2 / 2^23) in double; z_v = sigma * n + w * q(r(v))
 *   draft  n' = (sum of the 2 uniforms of lowbias32(x) - 1) * sqrt(6) with x from R_D;
 *     d_v = z_v + tau_b * n', tau_b = tau[0] for b < tau_split, else tau[1]. */
typedef struct {
    uint64_t seed;       /* target rows */
    uint64_t draft_seed; /* draft noise */
    float sigma;         /* scale of the target rows' noise */
    float alpha;         /* weight of the rank term, about -alpha ln(1 + rank) */
    float tau[2];        /* draft noise scale of sequences b < tau_split, and of the others */
    int32_t tau_split;
} psd_toy_lm;

/* The toy model's rows for one block: target rows device [B][gamma+1][V] at
 * positions start_pos[b] + s, and draft rows device [B][K][gamma][V] (nullable),
 * in params->dtype.  start_pos device [B] int64. */
psd_status psd_toy_logits(const psd_params *params, const psd_toy_lm *lm, int32_t batch, int32_t gamma,
                          const int64_t *start_pos, void *target_logits, void *draft_logits, hipStream_t stream);

/* Bytes of device scratch psd_generate needs: the block workspace, the block's
 * target and draft rows and the loop's state (lengths, starts, windows).  0 for
 * invalid arguments. */
size_t psd_generate_workspace_bytes(const psd_params *params, int32_t batch, int32_t gamma);

/* Generate n_pos tokens after each prompt with the toy model, block after block on
 * the device: toy rows -> psd_verify (drafts in the fused kernel, target_rows 1) ->
 * psd_advance.  The host reads one word (the active count) every check_every
 * blocks and stops when it is 0.  With use_graph != 0, check_every blocks are
 * captured once into a HIP graph on a stream of the call's own (ordered after the
 * work already on `stream`) and the graph is replayed.  Blocks the calling thread
 * until the texts are complete.
 *   text        device [B][text_stride] int32: prompts in [0, m) (m = ctx_window); out:
 *               the generated tokens in [m, m + n_pos)
 *   workspace   device, psd_generate_workspace_bytes(), 256-byte aligned
 *   out_blocks  host, nullable: blocks run (at most check_every - 1 past the last
 *               sequence's end)
 *   out_status  host, nullable: the error bits of all the blocks (0 = healthy)
 * Any top_k / top_p, mode and clock layout of params apply to every block. */
psd_status psd_generate(const psd_params *params, const psd_toy_lm *lm, int32_t batch, int32_t gamma, int32_t n_pos,
                        int32_t *text, int64_t text_stride, void *workspace, size_t workspace_bytes,
                        int32_t check_every, int32_t use_graph, int32_t *out_blocks, uint32_t *out_status,
                        hipStream_t stream);

/* ---- parity exports: the keyed randomness itself ---------------------------- */

/* Philox4x32-10 blocks: out[i][0..3] = Philox(ctr[i][0..3], key[i][0..1]).
 * ctr device [n][4] uint32, key device [n][2] uint32, out device [n][4] uint32. */
psd_status psd_philox(int32_t n, const uint32_t *ctr, const uint32_t *key, uint32_t *out, hipStream_t stream);

/* Context keys kappa = H(key, t[i], windows[i][0..m)) for n contexts.
 * t device [n] int64, windows device [n][m] int32 (oldest first, -1 = none),
 * out_kappa device [n][2] uint32.  Uses params->key and params->ctx_window. */
psd_status psd_context_keys(const psd_params *params, int32_t n, const int64_t *t, const int32_t *windows,
                            uint32_t *out_kappa, hipStream_t stream);

/* Clocks E_slot[token] in double for n (kappa, slot, token) triples under
 * params->clocks and params->vocab.  kappa device [n][2], slot device [n] int32,
 * token device [n] int32 (0 <= token < V), out device [n] double. */
psd_status psd_clock_values(const psd_params *params, int32_t n, const uint32_t *kappa, const int32_t *slot,
                            const int32_t *token, double *out, hipStream_t stream);

const char *psd_last_error(void); /* thread-local message of the last non-OK status */

/* Test hook: polls of a bounded wait before it gives up and sets error bit 0, for
 * the calls launched after it (process-wide; 0 restores the default, 2^22).  A
 * tiny limit makes waits give up on purpose while every kernel still runs to
 * completion, so the error path can be exercised from the host. */
void psd_set_spin_limit(uint32_t polls);
int32_t psd_abi_version(void);    /* PSD_ABI_VERSION */

#ifdef __cplusplus
}
#endif

#endif /* PSD_H */
