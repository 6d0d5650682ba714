/*
 * Entry points of the library that only the Python binding calls: forms of
 * the public calls (include/attnfuse.h) that take scratch memory.  They are not
 * part of the C ABI and may change with the binding.
 */
#ifndef AF_BINDING_H
#define AF_BINDING_H

#include <stddef.h>

#ifdef __cplusplus
extern "C" {
#endif

/* Bytes of scratch with which the forward of these sizes runs faster (the keys
 * rotated once into it), or 0 where it is better without.  extra: 1 with ALiBi
 * slopes or a bias; sparse_blocks: the active blocks of a block mask, 0 without
 * one. */
size_t af_fwd_workspace_bytes(int B, int H, int H_kv, int S, int D, int dtype, int rope, int mask, int window,
                              int norm, int extra, long long sparse_blocks);

/* Waves per workgroup (4 or 8) of the dense forward of these sizes where both
 * forms exist; rope: AF_ROPE_NONE for tiles that are not rotated in the loop;
 * bias: 0 without one, 1 where one row serves every query, 2 a row per query. */
int af_fwd_waves(int B, int H, int H_kv, int S, int D, int rope, int mask, int window, int bias);

/* attnfuse_fwd (bias == NULL, q_block_ptr == NULL), attnfuse_fwd_bias_norm or
 * attnfuse_fwd_blocksparse with RoPE on bf16 tensors, given
 * 2 * B * H_kv * S * D bytes of 16-byte aligned device scratch; same results. */
int af_fwd_ws(const void* Q, const void* K, const void* V, void* O, float* LSE, const int* q_block_ptr,
              const int* k_block_idx, const float* bias, long long bias_stride_b, long long bias_stride_h,
              long long bias_stride_q, int norm, void* workspace, size_t workspace_bytes,
              int B, int H, int H_kv, int S, int D, int dtype,
              int rope, float rope_theta, const float* rope_table, int rope_table_rows, int mask, int window,
              const float* alibi_slopes, float softmax_scale, void* stream);

/* attnfuse_bwd_blocksparse, told how long the mask's lists are: the 64-row
 * query tiles that the longest 128-key block of the mask (within the causal
 * range under a causal or window mask) visits, and those of all of them.  0:
 * not known, and one workgroup takes each key block. */
int af_bwd_blocksparse(const void* Q, const void* K, const void* V, const void* O, const void* dO,
                       const float* LSE, void* dQ, void* dK, void* dV,
                       const int* q_block_ptr, const int* k_block_idx,
                       const int* k_block_ptr, const int* q_block_idx, int longest_list, long long list_tiles,
                       void* workspace, size_t workspace_bytes,
                       int B, int H, int H_kv, int S, int D, int dtype,
                       int rope, float rope_theta, const float* rope_table, int rope_table_rows,
                       int mask, int window,
                       const float* alibi_slopes, float softmax_scale, void* stream);

/* The list lengths af_bwd_blocksparse takes, of a block mask [nb][nb] in host
 * memory (a byte per block, 0 or 1): {longest, all} without an elementwise mask,
 * then within the causal range. */
void af_col_tiles(const unsigned char* active, int nb, long long* lengths);

/* Workgroups that share a key block in the bf16 dK/dV pass of these sizes, given
 * partial_bytes of workspace for their partials; list_tiles < 0: without a block mask. */
int af_bwd_splits(int B, int H, int H_kv, int S, int D, int mask, int window, int longest_list, long long list_tiles,
                  size_t partial_bytes);

#ifdef __cplusplus
}
#endif

#endif
