// Internal launch interface between the C-ABI layer (abi.hip) and the kernel files.
// Every launcher assumes its arguments were validated by the C-ABI layer.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "bom.h"

namespace bom {

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// ---- residual ------------------------------------------------------------------------------
size_t residual_workspace_bytes(int64_t N, int64_t V, bom_dtype dt);
hipError_t launch_residual(const void* Z, bom_dtype dt, int N, int V, int64_t ldz, const int32_t* labels,
                           int32_t ignore_index, float* s, float* row_lse, int32_t* row_argmax, float* row_target,
                           void* R, int64_t ldr, float* loss, int32_t* n_valid, int32_t* flags, void* ws,
                           hipStream_t stream);

// Allocation-free residual: the device address of this device's fixed scratch array (looked up once per
// device, with that device current) of kResidualScratchBytes, which takes the workspace's place.
constexpr size_t kResidualScratchBytes = (size_t)BOM_RESIDUAL_SCRATCH_BYTES;
hipError_t residual_scratch(void** ptr);

// ---- EMA -----------------------------------------------------------------------------------
hipError_t launch_ema(float* q, const float* s, int64_t V, float beta1, float inv_bc1, float* q_hat,
                      hipStream_t stream);

// ---- head VJP --------------------------------------------------------------------------------
struct HeadVjpArgs {
    const void* H; int64_t ldh;
    const void* W; int64_t ldw;
    const void* R; int64_t ldr;       // residual rows R, or the logits Z when is_residual == 0
    int is_residual;
    const float* row_lse;             // [N], read when is_residual == 0
    bom_dtype dt;
    int N, d, V;
    const int32_t* labels; int32_t ignore_index;
    const float* q_hat; const float* s; const int32_t* n_valid; float lambda;
    void* dW; bom_dtype dw_dt; int64_t lddw; float dW_beta;   // dW and db in dw_dt (fp32 or bf16)
    void* db;
    void* dH; bom_dtype dh_dt; int64_t lddh;
    void* ws; size_t ws_bytes;
    size_t scratch_bytes = 0;   // fp32 dW and db of the same call that lie past the workspace of the products
};
// The second: with the panels of R that large products from the logits run on when the workspace holds them.
size_t head_vjp_workspace_bytes(int64_t N, int64_t d, int64_t V, bom_dtype dt, bom_dtype dw_dt);
size_t head_vjp_logits_workspace_bytes(int64_t N, int64_t d, int64_t V, bom_dtype dt, bom_dtype dw_dt);
hipError_t launch_head_vjp(const HeadVjpArgs& a, hipStream_t stream);

// fp32 operands: both products (and db) on the fp32 matrix instructions. dW is the sum of `sums` partial sums of equal
// k ranges, in order; `part` holds the sums of k ranges that go to units of their own.
size_t vjp_f32_workspace_bytes(int64_t N, int64_t d, int64_t V, int sums);
hipError_t launch_vjp_f32_products(const HeadVjpArgs& a, int sums, void* part, hipStream_t stream);
hipError_t launch_forward_f32(const float* H, int64_t ldh, const float* W, int64_t ldw, const float* b, int N, int d,
                              int V, float* Z, int64_t ldz, hipStream_t stream);

// ---- head telemetry (diagnostic) --------------------------------------------------------------
struct TeleArgs {
    const void* H; int64_t ldh; bom_dtype h_dt;
    const void* R; int64_t ldr; bom_dtype r_dt;
    int N, d, V;
    const int32_t* labels; int32_t ignore_index;
    const float* s; const float* q_hat; const int32_t* n_valid;
    float* MW; int64_t ldm; float* Mb;
    float beta1, one_minus_beta1, inv_bc;
    float* out;
    void* ws;
};
size_t head_telemetry_workspace_bytes(int64_t N, int64_t d);
hipError_t launch_head_telemetry(const TeleArgs& a, hipStream_t stream);

// ---- head forward (support) ---------------------------------------------------------------
hipError_t launch_head_forward(const void* H, int64_t ldh, const void* W, int64_t ldw, const void* b, bom_dtype dt,
                               int N, int d, int V, void* Z, int64_t ldz, hipStream_t stream);

// ---- update ----------------------------------------------------------------------------------
struct SegTable {
    int n;
    int64_t begin[BOM_MAX_SEGMENTS];
    int64_t end[BOM_MAX_SEGMENTS];
    float wd[BOM_MAX_SEGMENTS];
    float wd_default;
};
struct UpdateScalars {
    float lr, beta2, one_minus_beta2, eps, lambda, u_scale, inv_bc2;
    float clip_norm;      // > 0: global-norm clipping of the numerator
    const float* clip;    // device word with the clipping factor (written on the device), or null
    float* clip_stats;    // optional device [2]: the numerator's norm before clipping and the factor
    float beta1, one_minus_beta1, inv_bc1;   // AdamW's first moment (the comparison update)
};
size_t update_workspace_bytes(int64_t P, const bom_update_cfg* cfg);
hipError_t launch_update_dense(float* theta, float* v, const float* u, const float* h, int64_t P, const SegTable& segs,
                               UpdateScalars sc, void* ws, hipStream_t stream);
hipError_t launch_update_dense_bf16(uint16_t* theta, uint16_t* v, const uint16_t* u, const uint16_t* h, int64_t P,
                                    const SegTable& segs, UpdateScalars sc, void* ws, hipStream_t stream);
// Block-shared second moment: segments tiling [0, P) in order, each cut into blocks of blk[k] elements.
struct BlockSegs {
    int n;
    int64_t begin[BOM_MAX_SEGMENTS];
    int64_t len[BOM_MAX_SEGMENTS];
    int64_t blk[BOM_MAX_SEGMENTS];
    float wd[BOM_MAX_SEGMENTS];
};
int64_t blocks_count(const BlockSegs& b);
hipError_t launch_update_blocks(float* theta, float* v, const float* u, const float* h, int64_t P, const BlockSegs& bs,
                                UpdateScalars sc, void* ws, hipStream_t stream);
hipError_t launch_update_factored(float* theta, float* Rr, float* Cc, const float* u, const float* h, int64_t P,
                                  int64_t block_rows, int64_t block_cols, const SegTable& segs,
                                  const UpdateScalars& sc, void* ws, hipStream_t stream);
// AdamW (the comparison optimizer of the cost model): dense, or with the factored second moment for
// block_cols of 1024, 2048 or 4096.
hipError_t launch_adamw_dense(float* theta, float* m, float* v, const float* g, int64_t P, const SegTable& segs,
                              const UpdateScalars& sc, hipStream_t stream);
hipError_t launch_adamw_factored(float* theta, float* m, float* Rr, float* Cc, const float* g, int64_t P,
                                 int64_t block_rows, int64_t block_cols, const SegTable& segs, const UpdateScalars& sc,
                                 void* ws, hipStream_t stream);

}  // namespace bom
