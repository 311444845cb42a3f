/* eqlinear_block.h -- kernels of the equivariant encoder block around its
 * linear layers (inference).  Same library, dtypes, status codes and rules as
 * eqlinear.h: device pointers of 16-byte alignment (weight and bias: of their
 * element), the caller's stream, every argument checked before any launch, no
 * allocation, no synchronisation, bitwise reproducible. */
#ifndef EQLINEAR_BLOCK_H
#define EQLINEAR_BLOCK_H

#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

/* Layer norm of the encoder block over the C * T elements of each row:
 * y[r, c, t] = (x[r, c, t] - mean_r) / sqrt(var_r + eps) * weight[c] + bias[c],
 * var the mean squared deviation, all in fp32, rounded once.  x, y [rows, C, T],
 * weight, bias [C], one dtype.  A row must be whole 16-byte words and at most
 * 16 KB (EQL_ERR_UNSUPPORTED otherwise); rows = 0 is a no-op.  y overlaps no
 * input. */
int eqlinear_group_norm(const void* x, const void* weight, const void* bias, void* y, int64_t rows, int T, int C,
                        float eps, int dtype, void* stream);

/* Softmax attention of the encoder block: qkv [B, L, 3, heads, head_dim] (as
 * the qkv layer writes it), o [B, L, heads, head_dim],
 * o[b, q, h] = sum_k softmax_k(scale * <Q[b, q, h], K[b, k, h]>) V[b, k, h].
 * EQL_F16 and EQL_BF16, head_dim 32, 64 or 128, 1 <= L <= 256, scale > 0
 * (EQL_ERR_UNSUPPORTED for other sizes and fp32).  Scores and softmax in fp32,
 * the probabilities rounded once to the dtype, products accumulated in fp32.
 * B = 0 is a no-op. */
int eqlinear_attention(const void* qkv, void* o, int64_t B, int L, int heads, int head_dim, float scale, int dtype,
                       void* stream);

#ifdef __cplusplus
}
#endif

#endif /* EQLINEAR_BLOCK_H */
