// Host-side launch interface between the C ABI (mx_api.hip) and the kernels.
// All arguments have been validated by the caller.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace mxl {

// bf16 -> FP32 of a short vector (a bias), done by one more workgroup of a quantizer launch.
struct WidenJob {
    const uint16_t* src = nullptr;
    float* dst = nullptr;
    uint32_t count = 0;
};

// What is left of a column sum after the quantizer's pass: [blocks][cols] FP32 partials to be added up.
struct ColumnSumTail {
    const float* partials = nullptr;
    void* out = nullptr;       // cols values, FP32 or bf16 (the FP32 sum rounded to nearest even)
    uint32_t blocks = 0, cols = 0;
    int out_bf16 = 0;
};

struct QuantRowsParams {
    const void* src;
    bool bf16;
    int64_t rows, cols, ld;
    uint8_t* codes;
    uint8_t* scales;
    bool sr;
    bool floor_mode;
    uint64_t seed;
    uint32_t tensor_id;
    uint64_t index_base;
};

struct QuantTileParams {
    const void* src;
    bool bf16;
    int64_t rows, cols, ld;
    uint8_t* codes_t;
    uint8_t* scales_t;
    bool sr_t;
    uint32_t tensor_id_t;
    bool pre_quant;
    uint8_t* codes_row;
    uint8_t* scales_row;
    bool sr_row;
    uint32_t tensor_id_row;
    const uint8_t* row_codes_in;
    const uint8_t* row_scales_in;
    bool floor_mode;
    uint64_t seed;
    uint64_t index_base;
    const uint64_t* seed_dev = nullptr;   // device word that replaces `seed` when set
    int64_t src_rows = 0;                 // rows the source has (0: all); the rest up to `rows` count as zero
    void* col_sums = nullptr;             // [cols] column sums of the source (needs a source), FP32 or bf16, with
    bool col_sums_bf16 = false;
    float* col_sum_workspace = nullptr;   // column_sum_workspace_bytes(rows, cols) of scratch
};

// C[m x n] = A[m x k] . B[n x k]^T, operands packed MXFP4 along k.
struct GemmParams {
    const uint8_t* a_codes;
    const uint8_t* a_scales;
    const uint8_t* b_codes;
    const uint8_t* b_scales;
    int64_t m, n, k;
    void* c;
    bool c_bf16;
    int64_t ldc;
    void* workspace;
    int split_k;     // >= 1; > 1 needs workspace of split_k * m * n floats
    const float* bias = nullptr;   // n values added to every output row (needs n % 4 == 0), or null
    // fused GELU + 1x32 round_D quantizer of the output (needs bias, k % 128 == 0, k >= 512, no K split,
    // n % 32 == 0): codes [m x n/2], scale bytes [m x n/32]; gemm_takes_fused_quantizer() tells
    uint8_t* q_codes = nullptr;
    uint8_t* q_scales = nullptr;
    bool q_floor = false;
};
// Whether launch_gemm runs these sizes on the kernel that carries the fused output quantizer.
bool gemm_takes_fused_quantizer(int64_t m, int64_t n, int64_t k);

// What every caller's arguments must satisfy before a launch (MX_OK or an MX_ERR_* code), for the C interface and the
// native front ends alike: the kernels themselves rely on it.
int check_rows(const QuantRowsParams& p);
int check_ema(const QuantRowsParams& p, const float* ema, float beta, int update_ema);
int check_tile(const QuantTileParams& p);
int check_gemm(const GemmParams& p);                    // without the workspace, whose size the caller knows

hipError_t launch_quantize_rows(const QuantRowsParams& p, hipStream_t st);
// round_D rows of up to two contiguous tensors of any source types, and a vector to widen, in one launch.
hipError_t launch_quantize_rows_batch(const QuantRowsParams* p, int count, hipStream_t st, const WidenJob* widen = nullptr);
hipError_t launch_quantize_rows_e3m0(const QuantRowsParams& p, hipStream_t st);      // E3M0 elements (Table 7)
hipError_t launch_dequantize_e3m0(const uint8_t* codes, const uint8_t* scales, int64_t rows, int64_t cols,
                                  float* out, hipStream_t st);
hipError_t launch_ema_quantize(const QuantRowsParams& p, float* ema, float beta, int update_ema, hipStream_t st);
hipError_t launch_quantize_tile(const QuantTileParams& p, hipStream_t st);
size_t column_sum_workspace_bytes(int64_t rows, int64_t cols);
// Up to 4 tensors in one launch; they must share kind of source (FP32 and bf16 may be mixed where the rows round
// deterministically and no column sums are taken), roundings and scale rule.  finish_col_sums false: the caller adds up
// the column sums' partials itself (column_sum_tail), e.g. in the launch that reduces a K split.
hipError_t launch_quantize_tile_batch(const QuantTileParams* jobs, int count, hipStream_t st, const WidenJob* widen = nullptr,
                                      bool finish_col_sums = true);
// Workgroups (of four waves) that one tensor's launch has (for tests of the rule); src: 0 FP32, 1 bf16, 2 packed codes.
uint32_t tile_workgroups(int64_t rows, int64_t cols, int src, bool row_sr, bool t_sr);
ColumnSumTail column_sum_tail(const QuantTileParams& q);
hipError_t launch_column_sum_finish(const ColumnSumTail& t, hipStream_t st);
hipError_t launch_dequantize(const uint8_t* codes, const uint8_t* scales, int64_t rows, int64_t cols,
                             float* out, hipStream_t st);

struct OscillationParams {
    const void* w;
    bool bf16;
    int64_t rows, cols, ld;
    const uint8_t* codes;
    const uint8_t* scales;
    float* w_prev;
    uint8_t* codes_prev;
    uint8_t* scales_prev;
    float* dist_w;
    float* dist_q;
    int init;
};
hipError_t launch_oscillation(const OscillationParams& p, hipStream_t st);
hipError_t launch_ramping_factor(const float* dist_w, const float* dist_q, int64_t count, float k1, int k2,
                                 int n_max, int32_t* factor, hipStream_t st);

struct ConfidenceParams {
    const void* w;
    bool bf16;
    int64_t rows, cols, ld;
    int floor_mode;
    float* conf;            // may be null
    uint64_t* hist;         // may be null
    int bins;
};
constexpr int CONFIDENCE_MAX_BINS = 1024;
hipError_t launch_confidence(const ConfidenceParams& p, hipStream_t st);

struct RateParams {
    const void* x;
    bool bf16;
    int64_t rows, cols, ld;
    float* x_prev;
    int init;
    double* partial;        // rate_workspace_bytes() of scratch
    double* result;         // 3 doubles
};
size_t rate_workspace_bytes();
hipError_t launch_rate_of_change(const RateParams& p, hipStream_t st);

struct RampingAdamwParams {
    float* w;
    const void* grad;
    bool grad_bf16;
    int64_t count;          // multiple of 4
    float* m;
    float* v;
    float* g_acc;           // null iff factor is null
    const int32_t* factor;  // null: plain AdamW
    int32_t* acc_steps;     // null iff factor is null
    int32_t* updates;
    float lr, beta1, beta2, eps, weight_decay;
};
hipError_t launch_ramping_adamw(const RampingAdamwParams& p, hipStream_t st);
// Any number of tensors (ADAM_BATCH_MAX per launch), all with factors or all without, the first one's hyper-parameters.
constexpr int ADAM_BATCH_MAX = 32;
hipError_t launch_ramping_adamw_batch(const RampingAdamwParams* p, int count, hipStream_t st);

// One step of a detection window for dense FP32 weights whose rows are a multiple of 32 long.
struct WindowTensor {
    float* w;
    const void* grad;          // null: the weight stands still
    float* m;
    float* v;
    int32_t* updates;
    float* g_acc;
    int32_t* acc_steps;
    float* w_prev;
    float* dist_w;
    float* dist_q;
    uint8_t* codes_prev;
    uint8_t* scales_prev;
};
struct RampingWindowParams {
    float lr, beta1, beta2, eps, weight_decay;
    bool opens, floor_mode;
};
constexpr int WINDOW_BATCH_MAX = 24;
hipError_t launch_ramping_window_batch(const RampingWindowParams& p, const WindowTensor* tensors, const int64_t* counts,
                                       const bool* grad_bf16, int count, hipStream_t st);

hipError_t launch_calibration_copy(void* dst, const void* src, size_t bytes, hipStream_t st);

// Register-resident MFMA loop (calibration of the matrix pipe's sustained rate on given operand bytes).
size_t calibration_mfma_operand_bytes();
hipError_t launch_calibration_mfma(const uint8_t* operands, int workgroups, int iterations, float* sink, hipStream_t st);

// Number of K-splits the product will use for these sizes (1 = none).
int gemm_split_k(int64_t m, int64_t n, int64_t k);
// Kernel that a product, or one with the fused output quantizer, is planned on (for tests of the rules).
const char* gemm_kernel_name(int64_t m, int64_t n, int64_t k, bool fused);
// tail: column sums to finish as well (in the K split's reduction where there is one, else in a launch of their own).
hipError_t launch_gemm(const GemmParams& p, hipStream_t st, const ColumnSumTail* tail = nullptr);
// C[m x n] = Q(x[m x k]) . Q(w[n x k])^T + bias with round_D row quantizers, in one launch that keeps no codes; dense rows,
// 16-byte aligned x, w and bias, n and k multiples of 32.  Worth it, and allowed, where linear_fits_one_launch says so.
struct QuantizedLinearParams {
    const void* x;
    const void* w;
    const void* bias;          // n values or null
    bool x_bf16, w_bf16, bias_bf16, floor_mode;
    int64_t m, n, k;
    void* c;
    bool c_bf16;
};
// captured: the stream is recording a graph.  The codes and sums are those of the separate kernels either way.
bool linear_fits_one_launch(int64_t m, int64_t n, int64_t k, bool bias_bf16, bool captured);
hipError_t launch_quantized_linear(const QuantizedLinearParams& p, hipStream_t st);
// Two independent products, in one launch where that pays; the results of launch_gemm(x) and launch_gemm(w, tail), bit for bit.
hipError_t launch_gemm_pair(const GemmParams& w, const GemmParams& x, hipStream_t st, const ColumnSumTail* tail = nullptr);
// Whether it makes one launch of them, given a workspace for each that splits K; otherwise they run x, then w, and may share one.
bool gemm_pair_fits_one_launch(const GemmParams& w, const GemmParams& x);

}  // namespace mxl
