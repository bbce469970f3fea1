// Row kernels of the decoder around the attention (chunk_loop.py): launched through these C functions by the extension
// module of the binding.  All tensors are contiguous; dtype is a seco_dtype; the functions return a seco_status.
#pragma once
#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif
// x_out = x + y (y NULL: x_out is not written), h = round(x_out * rstd) * gain, rstd = 1 / sqrt(mean(x_out^2) + 1e-6)
int dec_add_rmsnorm(int dtype, const void* x, const void* y, const void* gain, void* x_out, void* h, float* rstd,
                    int64_t rows, int64_t d, void* stream);
// the same for the rows token[r] of a table of v rows, which go to x_out; a token outside [-v, v) gives NaN, a negative one counts from the end
int dec_embed_rmsnorm(int dtype, const void* table, const int64_t* token, const void* gain, void* x_out, void* h, float* rstd,
                      int64_t rows, int64_t d, int64_t v, void* stream);
// ... and *outside (NULL: nothing) becomes 1 if there is such a token; else it stays as it is
int dec_embed_rmsnorm_checked(int dtype, const void* table, const int64_t* token, const void* gain, void* x_out, void* h, float* rstd,
                              int64_t rows, int64_t d, int64_t v, float* outside, void* stream);
// d_x = d_in + gradient of the norm at x (d_in NULL: the gradient alone; d_x may be d_in or d_h);
// gain_part[blocks, d] fp32 += per-workgroup sums of the gain's gradient, blocks = DEC_GAIN_BLOCKS
#define DEC_GAIN_BLOCKS 256
int dec_rmsnorm_bwd(int dtype, const void* x, const void* gain, const float* rstd, const void* d_h, const void* d_in,
                    void* d_x, float* gain_part, int64_t rows, int64_t d, void* stream);
// sums[n, d] = parts[n, DEC_GAIN_BLOCKS, d] summed over the blocks in a fixed order; rounded (NULL: not written): the same in dtype
int dec_gain_sums(int dtype, const float* parts, float* sums, void* rounded, int64_t n, int64_t d, void* stream);
// src [rows, a + b + c bytes] -> a, b, c, each contiguous; sizes are multiples of 16 bytes
int dec_split_columns(const void* src, void* a, void* b, void* c, int64_t rows, int64_t bytes_a, int64_t bytes_b, int64_t bytes_c,
                      void* stream);
int dec_silu(int dtype, const void* u, void* a, int64_t n, void* stream);
int dec_silu_bwd(int dtype, const void* u, void* d_a, int64_t n, void* stream);   // d_a <- d_a * silu'(u)
// loss[r] = logsumexp(logits[r]) - logits[r][target[r]] (loss non-NULL), or logits <- softmax - onehot (loss NULL);
// a target of -100 gives loss 0 and gradient 0, any other target outside [0, v) NaN
int dec_cross_entropy(int dtype, void* logits, const int64_t* target, float* loss, int64_t rows, int64_t v, void* stream);
// both: the loss (loss non-NULL), and logits <- softmax - onehot; the same values
int dec_cross_entropy_both(int dtype, void* logits, const int64_t* target, float* loss, int64_t rows, int64_t v, void* stream);
// grad[token[r]] += d_x[r] for every row r; the rows of one token are added in ascending order by one workgroup
int dec_embedding_bwd(int dtype, const void* d_x, const int64_t* token, void* grad, int64_t rows, int64_t d, int64_t v,
                      void* stream);
// A layer's joint projection qkv [B, C, (Hq + 2 Hkv) D] and rows row0 .. row0 + C of its cache (k, v: the type of qkv) or, with
// `inverse`, of its fp32 gradient buffers, both [B, Hkv, *, D] with kv_stride: queries rotated (back) in place, keys rotated and
// values copied to the cache, or gK (rotated back) and gV to the key and value columns; what rope_rotate with
// kv_append_rope, or kvgrad_readout_rope with rope_rotate, compute, bit for bit, in one launch.  D as there: bf16 128, fp32 a multiple of 8 up to 256
int dec_rope_qkv(int dtype, int inverse, void* qkv, void* k, void* v, const int64_t* kv_stride, int64_t B, int64_t Hq, int64_t Hkv,
                 int64_t C, int64_t D, int64_t row0, float base, void* stream);

// bf16 matrix products with fp32 accumulation, row-major with leading dimensions in elements (gemm_bf16.hip):
//   NN: C[M,N] = A[M,K] B[K,N]     NT: C[M,N] = A[M,K] B[N,K]^T     TN: C[M,N] = A[K,M]^T B[K,N]
// Epilogues: STORE; ADD (TN): C += the product; SILU (NN): C = the product, C2 = silu(C);
// SILU_BWD (NT): C = the product times silu'(C2).  Operands start on 16-byte boundaries.
enum { DEC_GEMM_NN = 0, DEC_GEMM_NT = 1, DEC_GEMM_TN = 2 };
enum { DEC_GEMM_STORE = 0, DEC_GEMM_ADD = 1, DEC_GEMM_SILU = 2, DEC_GEMM_SILU_BWD = 3 };
int dec_gemm_supported(int form, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, int64_t ldc);   // 1 / 0
int dec_gemm(int form, int epilogue, const void* a, const void* b, void* c, void* c2, int64_t M, int64_t N, int64_t K,
             int64_t lda, int64_t ldb, int64_t ldc, void* stream);
// Both gradients of y[M,n] = x[M,K] w[K,n], contiguous: dx[M,K] = dy w^T (u non-NULL: times silu'(u)), dw += x^T dy; what
// dec_gemm computes for either, bit for bit, in one launch where that pays.  No output may overlap an operand of the other.
int dec_gemm_grads(const void* dy, const void* w, void* dx, void* u, const void* x, void* dw, int64_t M, int64_t K, int64_t n, void* stream);
// the same with dw = x^T dy
int dec_gemm_first_grads(const void* dy, const void* w, void* dx, void* u, const void* x, void* dw, int64_t M, int64_t K, int64_t n, void* stream);
// The joint projection qkv[B C, (Hq + 2 Hkv) 128] = h[B C, K] w and what dec_rope_qkv makes of it, bit for bit, in one launch up to tiles of
// 64 rows; the key and value columns of qkv may be written or not
int dec_gemm_qkv(const void* h, const void* w, void* qkv, void* k, void* v, const int64_t* kv_stride, int64_t B, int64_t Hq, int64_t Hkv,
                 int64_t C, int64_t K, int64_t row0, float base, void* stream);
#ifdef __cplusplus
}
#endif
