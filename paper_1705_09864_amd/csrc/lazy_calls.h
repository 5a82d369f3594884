// Calls of include/bmx.h for the native module of the Python binding, which allocates a workspace
// only when one is needed: as the call of the same name, but the workspace may be null, and
// BMX_ERR_WORKSPACE then means that nothing was launched and that the call needs it.  (Finding a block in
// the caching allocator and giving it back costs 0.45 us of a call's 3.5 us on the host.)
#pragma once
#include <stddef.h>
#include <stdint.h>

extern "C" {
int bmx_lazy_binary_fc(const float* x, int64_t ldx, const uint64_t* Wp, int64_t ldw_w, const float* alpha, int batch,
                       int in_features, int out_features, int32_t* out_i32, float* out_f32, int64_t ldo, void* workspace,
                       size_t workspace_bytes, void* stream);
int bmx_lazy_binary_conv2d(const float* x, int N, int C, int H, int W, const uint64_t* Wp, int O, int KH, int KW,
                           int stride, int pad, const float* alpha, int32_t* out_i32, float* out_f32, void* workspace,
                           size_t workspace_bytes, void* stream);
int bmx_lazy_xnor_gemm_w32(const uint32_t* A, int64_t lda_dw, const uint32_t* B, int64_t ldb_dw, int32_t* C, int64_t ldc,
                           int M, int N, int K, void* workspace, size_t workspace_bytes, void* stream);
int bmx_lazy_binary_conv2d_bits(const uint64_t* xp, int N, int C, int H, int W, const uint64_t* Wp, int O, int KH, int KW,
                                int stride, int pad, const float* alpha, const float* thr, uint64_t* out_xp, int out_pad,
                                void* workspace, size_t workspace_bytes, void* stream);
int bmx_lazy_quant_gemm(const float* a, int64_t lda, int bits_a, const float* w, int64_t ldw, int bits_w, int M, int N,
                        int K, int32_t* out_i32_scaled, float* out_f32, int64_t ldo, void* workspace,
                        size_t workspace_bytes, void* stream);
}
