// The kernel launchers that the runtime calls beside the C ABI's: one
// declaration for the runtime, for the sources that define them and for the
// stand-ins of a host-only build, so that a signature that drifts does not link.
#pragma once
#include <hip/hip_runtime_api.h>

#include "../../include/rb.h"

// kernels.hip: reads a buffer on the stream, leaving only its clean lines in the caches
void rb_scrub_caches(hipStream_t stream, const void* buf, size_t bytes, unsigned* sink);
// gemm_f32_split.hip: one layer of an fp32 model on split weights, which hold W times 2^w_exp (X's rows gathered
// when src is given; the output through the row map when out_rows is)
rb_status rb_gemm_f32_split(hipStream_t s, const float* X, int ldx, const int64_t* src, int src_stride,
                            int64_t src_len, int* err, const void* Wp, int w_exp, const float* b, float* Y, int ldy,
                            int M, int N, int K, int act, const rb_k_row* skip_rows, int skip_T,
                            const rb_k_row* out_rows, int d_out, float* out);
// gemm_f32_split.hip: split weights, W [N, K] times scale, [Np, Kp] zero padded
rb_status rb_split_f32_weights(hipStream_t s, const float* W, int N, int K, int Np, int Kp, float scale, void* Wp);
// kernels.hip: rb_k_route and rb_k_embbag, with the ends of every row's bags passed from one to the other
extern "C" rb_status rb_route_bags(void* stream, int32_t kind, const rb_k_batch* batches, int32_t n_batches,
                                   const rb_k_req* reqs, int32_t n_reqs, const int32_t* lens, int64_t lens_len,
                                   int32_t d_in, int32_t d_out, int32_t n_tables, rb_k_row* rows, int32_t n_rows_total,
                                   int64_t out_len, int32_t* ends, int32_t fill, int32_t max_rows, int32_t* err);
extern "C" rb_status rb_embbag_ends(void* stream, const rb_k_row* rows, int32_t n_rows_total, const int32_t* lens,
                                    const int32_t* ends, const int32_t* ids, int64_t ids_len,
                                    const void* const* tables, int32_t n_tables, int64_t table_rows, int32_t emb_dim,
                                    const float* dense, int32_t n_dense, void* X, int32_t ldx, float pad, int32_t* err);
// kernels.hip: the arena offset of every packed token row
rb_status rb_token_rows(hipStream_t s, const rb_k_row* rows, int n_slots, int T, int64_t dense_len, int d_in,
                        int64_t* src, int64_t n_src, int* err);
// kernels.hip: the per-device address of the static scratch array (set up once
// per device; nullptr before that succeeded)
rb_status rb_static_scratch_setup(int device);
void* rb_static_scratch(int device);
