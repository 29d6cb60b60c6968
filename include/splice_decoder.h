/*
 * splice_decoder.h -- what lies between the weight products of a decode pass
 * around the spliced attention (paper Algorithm 1): norms, rotary embedding,
 * gated activation, residual stream, language-model head and argmax of a
 * pre-norm decoder with bf16 weights, one row per sweep cell.
 * decode.SweepDecoder calls these between its products and splice_decode_step.
 *
 * Each entry rounds where the same expression written out in PyTorch
 * operations rounds (bf16 product outputs, fp32 in between), so the values it
 * hands to the next product are those, bit for bit.  Pointers are device
 * memory, dense and 16-byte aligned, unless said otherwise; work is enqueued
 * on `stream`.  Statuses are splice_status; SPLICE_EUNSUPPORTED marks sizes an
 * entry does not take.
 */
#ifndef SPLICE_DECODER_H
#define SPLICE_DECODER_H

#include "splice_attn.h"

#ifdef __cplusplus
extern "C" {
#endif

/* x += delta (assign: x = delta), sq = x * x: n values, a multiple of 8; delta bf16. */
SPLICE_API int32_t splice_decoder_residual(float *x, const void *delta, float *sq, int64_t n, int32_t assign,
                                           void *stream);

/*
 * h = bf16(x * rsqrt(mean_sq[row] + eps) * gain): x [rows][d], gain bf16 [d], d a multiple of 8; h [rows][d], or
 * packed (d a multiple of 32) as splice_decoder_head reads it, [d / 32][ceil(rows / 16)][16][32].
 */
SPLICE_API int32_t splice_decoder_norm(const float *x, const float *mean_sq, const void *gain, void *h, int32_t rows,
                                       int32_t d, float eps, int32_t packed, void *stream);

/*
 * splice_decoder_residual, the mean of the squares and splice_decoder_norm at once, d at most
 * SPLICE_ADD_NORM_MAX_D: h plain, h_packed packed, either may be NULL.  The
 * squares are added in the order in which PyTorch adds rows of 256 to 7680
 * values when there are at least eight; for other sizes the mean is as accurate
 * but may differ in its last bit.
 */
#define SPLICE_ADD_NORM_MAX_D 8192
SPLICE_API int32_t splice_decoder_add_norm(float *x, const void *delta, const void *gain, void *h, void *h_packed,
                                           int32_t rows, int32_t d, float eps, int32_t assign, void *stream);

/*
 * tab [rows][head_dim / 2] = (cos, sin) of position * theta^(-2 i / head_dim),
 * the angle computed in 64 bits.  Positions: pos (device, rows doubles), or
 * with pos == NULL prompt_len + max(step, 0) of the host int32 cell_step.
 */
SPLICE_API int32_t splice_decoder_rope_table(float *tab, const double *pos, const int32_t *cell_step, int32_t rows,
                                             int32_t head_dim, int32_t prompt_len, double theta, void *stream);

/* Rotates q [rows][n_q][head_dim] and k [rows][n_kv][head_dim] (bf16) in place, pairs (i, i + head_dim / 2). */
SPLICE_API int32_t splice_decoder_rope(void *q, void *k, const float *tab, int32_t rows, int32_t n_q, int32_t n_kv,
                                       int32_t head_dim, void *stream);

/* dst = bf16(src), [rows][d], d a multiple of 8 (packed: of 32, and packed as splice_decoder_norm's h). */
SPLICE_API int32_t splice_decoder_round(const float *src, void *dst, int32_t rows, int32_t d, int32_t packed,
                                        void *stream);

/* act = bf16(bf16(silu(gate)) * up), bf16, [rows][d] as splice_decoder_round; act may be gate unless packed. */
SPLICE_API int32_t splice_decoder_silu(const void *gate, const void *up, void *act, int32_t rows, int32_t d,
                                       int32_t packed, void *stream);

/*
 * y [rows][n] = bf16(x . w [k][n]), bf16, x packed, fp32 sums in the order of k: k a multiple of 128, n of 8.
 * splice_decoder_product_takes: whether a pass uses it (1) or leaves the product to the library (0).
 */
SPLICE_API int32_t splice_decoder_product_takes(int32_t rows, int32_t k, int32_t n);
SPLICE_API int32_t splice_decoder_product(const void *x, const void *w, void *y, int32_t rows, int32_t k, int32_t n,
                                          void *stream);

/*
 * logits [rows][vocab] = float(bf16(h . w [d][vocab])), bf16 inputs, h packed
 * (splice_decoder_norm), fp32 sums: 1..SPLICE_MAX_CELLS rows, d a multiple of
 * 32, vocab of 8.  scratch: splice_decoder_head_bytes bytes (may be 0) on the
 * current device.  splice_decoder_head_takes: whether a pass uses it (1) or
 * leaves the head to the library (0).
 */
SPLICE_API int32_t splice_decoder_head_takes(int32_t rows, int32_t d, int32_t vocab);
SPLICE_API int64_t splice_decoder_head_bytes(int32_t rows, int32_t d, int32_t vocab);
SPLICE_API int32_t splice_decoder_head(const void *h, const void *w, float *logits, int32_t rows, int32_t d,
                                       int32_t vocab, void *scratch, size_t scratch_bytes, void *stream);

/*
 * tokens[r] = the lowest index of the largest of logits[r][0..vocab) (a NaN
 * counts as the largest).  scratch: rows * SPLICE_ARGMAX_PARTS * 8 bytes.
 * logits aligned to 4 bytes, tokens and scratch to 8.
 */
#define SPLICE_ARGMAX_PARTS 64
SPLICE_API int32_t splice_decoder_argmax(const float *logits, int32_t rows, int32_t vocab, int64_t *tokens,
                                         void *scratch, void *stream);

#ifdef __cplusplus
}
#endif

#endif /* SPLICE_DECODER_H */
