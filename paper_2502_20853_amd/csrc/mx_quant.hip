// MXFP4 quantizer kernels for gfx950: streaming, no matrix cores (the fused
// tile kernel is bound by the vector ALUs, the others by memory and launch).
//
//  quantize_rows_kernel   1x32 groups along the columns (Q1, Q2, Q3 of Eqs. 3-4)
//  quantize_tile_kernel   32x1 groups stored transposed (Q4, Q5, Q6 of Eqs. 4-5),
//                         optionally fused with the 1x32 quantizer of the same
//                         source (one read of the tensor) and with double
//                         quantization (Sec. 3.3)
//  ema_quantize_kernel    Q-EMA (Eq. 8, Algorithm 1)
//  oscillation_kernel     trajectory lengths dist_W, dist_Q of Q-Ramping (Sec. 6.1)
//  ramping_factor_kernel  amplification factor N_w of Algorithm 2
//  confidence_kernel      quantization confidence per element and its histogram (Sec. 4.2)
//  rate_partial_kernel,   one term of the rate of change of a tensor (Sec. 4.1): FP64 sums of
//  rate_finish_kernel     squares, reduced in a fixed order
//  dequantize_kernel      test aid
//
// Work split: one lane owns 8 consecutive elements of a row (one 16-byte bf16
// load, one Philox call for its 8 rounding decisions, one 4-byte store of 8
// codes); 4 neighbouring lanes form a 1x32 group and reduce |x| with DPP.
#include "mx_device.hpp"
#include "mx_launch.hpp"

#include <algorithm>
#include <type_traits>

using namespace mxd;

namespace {

constexpr int ROWS_UNROLL = 4;       // 8-element chunks per lane in quantize_rows_kernel
constexpr int ROWS_THREADS = 256;

struct RowsArgs {
    const void* src;
    uint8_t* codes;
    uint8_t* scales;
    float* ema;            // Q-EMA only
    int64_t ld;            // elements
    uint32_t cpr;          // 8-element chunks per row (cols / 8)
    uint32_t total;        // rows * cpr
    int contiguous;        // ld == cols
    int floor_mode;
    uint32_t k0, k1, tensor_id;
    uint64_t base_blk;     // index_base >> 3
    float beta;
    int update_ema;
};

// Rounding mode of the integer forms (see mx_device.hpp); round_D of E2M1 goes through the conversion instructions, in
// any mode.
template <bool SR>
__device__ __forceinline__ void set_round_mode_for()
{
    if (SR) f32_round_toward_plus_inf();
    else    f32_round_toward_minus_inf();
}

// round_S codes of eight elements of a row, low nibble first, with sr_terms() of the block, in the rounding mode of round_S.
template <bool FLOOR, typename RAW>
__device__ __forceinline__ uint32_t sr_codes8(const RAW& x, uint32_t byte, const U8& rnd)
{
    const int e = grid_exponent(byte);
    uint32_t g[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) g[t] = sr_grid<FLOOR>(element_of(x, t), e, rnd.w[t]);
    uint32_t p = pack_grid<0>(g[0], g[0], g[1]);
    p = pack_grid<1>(p, g[2], g[3]);
    p = pack_grid<2>(p, g[4], g[5]);
    return pack_grid<3>(p, g[6], g[7]);
}

// The 1x32 quantizer with E3M0 elements (format ablation, Table 7): same work split as
// quantize_rows_kernel, the element codec one bit higher in the FP32 layout.
template <typename SrcT, bool SR, bool FLOOR>
__global__ __launch_bounds__(ROWS_THREADS) void quantize_rows_e3m0_kernel(RowsArgs a)
{
    set_round_mode_for<SR>();
    const SrcT* src = static_cast<const SrcT*>(a.src);
    for (uint32_t q = blockIdx.x * ROWS_THREADS + threadIdx.x; q < a.total; q += gridDim.x * ROWS_THREADS) {
        // a.total is a multiple of 4 and a quad starts at a multiple of 4: the four lanes of a group stay together
        int64_t off;
        if (a.contiguous) {
            off = (int64_t)q * 8;
        } else {
            uint32_t r = q / a.cpr;
            off = (int64_t)r * a.ld + (int64_t)(q - r * a.cpr) * 8;
        }
        const F8 x = load8(src + off);
        const uint32_t byte = scale_byte_e3m0(quad_max(amax_bits8(x)), FLOOR);
        const int e = grid_exponent_e3m0(byte);
        U8 rnd;
        if (SR) rnd = sr_addends_e3m0(a.base_blk + q, a.tensor_id, a.k0, a.k1);
        uint32_t packed = 0;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            uint32_t c = SR ? sr_code_e3m0<FLOOR>(x.v[t], e, rnd.w[t]) : rtn_code_e3m0<FLOOR>(x.v[t], e);
            packed |= c << (4 * t);
        }
        reinterpret_cast<uint32_t*>(a.codes)[q] = packed;
        if ((threadIdx.x & 3) == 0) a.scales[q >> 2] = (uint8_t)byte;
    }
}

// round_D is bound by memory: 50432 x 3072 bf16 in 60 us, 6.5 TB/s, FP32 in 132, 5.3 TB/s.  round_S of bf16 by the random
// numbers: 71 to 75 us, 5.2 to 5.5 TB/s (80 to 89 with all rounds of Philox on the vector units); of FP32 by memory, 133 us.  At
// 25216 x 1536 bf16 16 to 17 and 22 to 23 us.
template <typename SrcT, bool SR, bool FLOOR, bool WIDE>
__global__ __launch_bounds__(ROWS_THREADS) void quantize_rows_kernel(RowsArgs a)
{
    if (SR) f32_round_toward_plus_inf();
    using Blk = std::conditional_t<WIDE, uint64_t, uint32_t>;
    const SrcT* src = static_cast<const SrcT*>(a.src);
    const uint32_t q0 = blockIdx.x * (ROWS_THREADS * ROWS_UNROLL) + threadIdx.x;
    Raw8<SrcT> x[ROWS_UNROLL];
    bool ok[ROWS_UNROLL];
#pragma unroll
    for (int u = 0; u < ROWS_UNROLL; ++u) {
        uint32_t q = q0 + u * ROWS_THREADS;
        ok[u] = q < a.total && q >= q0;
        x[u] = Raw8<SrcT>{};
        if (ok[u]) {
            int64_t off;
            if (a.contiguous) {
                off = (int64_t)q * 8;
            } else {
                uint32_t r = q / a.cpr;
                off = (int64_t)r * a.ld + (int64_t)(q - r * a.cpr) * 8;
            }
            x[u] = load_raw8(src + off);
        }
    }
#pragma unroll
    for (int u = 0; u < ROWS_UNROLL; ++u) {
        uint32_t q = q0 + u * ROWS_THREADS;
        const uint32_t byte = row_scale_byte<FLOOR>(x[u]);
        uint32_t packed;
        if constexpr (SR) packed = sr_codes8<FLOOR>(x[u], byte, sr_terms(sr_counter((Blk)(a.base_blk + q), a.k1), (uint32_t)(a.base_blk >> 32), a.tensor_id, a.k0, a.k1));
        else              packed = rtn_codes8(x[u], byte);
        if (ok[u]) {
            reinterpret_cast<uint32_t*>(a.codes)[q] = packed;
            if ((threadIdx.x & 3) == 0) a.scales[q >> 2] = (uint8_t)byte;
        }
    }
}

// round_D rows of up to two tensors (the activation and the weight of a forward pass that needs no column groups), each
// with its own source type, and a bias to widen, in one launch: at the sizes of serving a launch costs more than
// its work.  The body is quantize_rows_kernel's for contiguous sources.
struct RowsBatch {
    RowsArgs job[2];
    int bf16[2];
    uint32_t first1;       // first workgroup of the second job
    mxl::WidenJob widen;
};

template <bool FLOOR, int UNROLL>
__global__ __launch_bounds__(ROWS_THREADS) void quantize_rows_batch_kernel(RowsBatch b)
{
    if (b.widen.count != 0u && blockIdx.x == gridDim.x - 1u) {
        for (uint32_t i = threadIdx.x; i < b.widen.count; i += ROWS_THREADS) b.widen.dst[i] = __uint_as_float((uint32_t)b.widen.src[i] << 16);
        return;
    }
    const int j = blockIdx.x >= b.first1 ? 1 : 0;
    const RowsArgs& a = b.job[j];
    const uint32_t q0 = (blockIdx.x - (j ? b.first1 : 0u)) * (ROWS_THREADS * UNROLL) + threadIdx.x;
    auto run = [&](auto tag) {
        using SrcT = decltype(tag);
        const SrcT* src = static_cast<const SrcT*>(a.src);
        Raw8<SrcT> x[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const uint32_t q = q0 + u * ROWS_THREADS;
            x[u] = Raw8<SrcT>{};
            if (q < a.total) x[u] = load_raw8(src + (size_t)q * 8);
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const uint32_t q = q0 + u * ROWS_THREADS;
            const uint32_t byte = row_scale_byte<FLOOR>(x[u]);
            const uint32_t packed = rtn_codes8(x[u], byte);
            if (q < a.total) {
                reinterpret_cast<uint32_t*>(a.codes)[q] = packed;
                if ((threadIdx.x & 3) == 0) a.scales[q >> 2] = (uint8_t)byte;
            }
        }
    };
    if (b.bf16[j]) run(uint16_t{});
    else           run(float{});
}

template <typename SrcT>
__global__ __launch_bounds__(ROWS_THREADS) void ema_quantize_kernel(RowsArgs a)
{
    const SrcT* src = static_cast<const SrcT*>(a.src);
    const uint32_t q = blockIdx.x * ROWS_THREADS + threadIdx.x;
    const bool ok = q < a.total;
    F8 w = zero8(), e = zero8();
    int64_t off = 0;
    if (ok) {
        if (a.contiguous) {
            off = (int64_t)q * 8;
        } else {
            uint32_t r = q / a.cpr;
            off = (int64_t)r * a.ld + (int64_t)(q - r * a.cpr) * 8;
        }
        w = load8(src + off);
        if (a.update_ema != 2) e = load8(a.ema + off);
    }
    if (a.update_ema == 1) {
        const float omb = __fsub_rn(1.0f, a.beta);
#pragma unroll
        for (int t = 0; t < 8; ++t) e.v[t] = __fmaf_rn(a.beta, e.v[t], __fmul_rn(omb, w.v[t]));
    } else if (a.update_ema == 2) {
        e = w;
    }
    uint32_t m = quad_max(amax_bits8(w));
    uint32_t byte = scale_byte(m, a.floor_mode);
    float inv = inv_scale(byte);
    uint32_t packed = 0;
#pragma unroll
    for (int t = 0; t < 8; ++t)
        packed |= round_ema(w.v[t] * inv, e.v[t] * inv, a.floor_mode,
                            (__float_as_uint(w.v[t]) & 0x7FFFFFFFu) == 0u) << (4 * t);
    if (ok) {
        if (a.update_ema != 0) {
            float4* p = reinterpret_cast<float4*>(a.ema + off);
            p[0] = make_float4(e.v[0], e.v[1], e.v[2], e.v[3]);
            p[1] = make_float4(e.v[4], e.v[5], e.v[6], e.v[7]);
        }
        reinterpret_cast<uint32_t*>(a.codes)[q] = packed;
        if ((threadIdx.x & 3) == 0) a.scales[q >> 2] = (uint8_t)byte;
    }
}

// ---------------------------------------------------------------------------
// Transposed / fused quantizer.
//
// A workgroup of 4 waves owns a 128 x 128 macro tile of the source (128 x 64 for small tensors and for the last tiles of
// others: tile_tail); with column sums, and for large FP32 sources (tile_waves), it has 8 waves and 256 rows.
// Wave w owns rows [32w, 32w+32) of it and walks over its 32 x 64 tiles.  The grid is one-dimensional over the macro tiles in row-major order.
// Inside a tile, lane l holds rows 4*(l/8)+j (j = 0..3) x columns 8*(l%8)+t (t = 0..7):
//   - each load instruction reads 8 full rows of 64 elements,
//   - a 1x32 row group is 4 neighbouring lanes (DPP quad reduction),
//   - a 32x1 column group is 4 registers x 8 lanes (l/8 = 0..7) of one column.
// The 32 elements of a lane stay in registers through both quantizers.  Codes and scale
// bytes are collected in LDS and written out at the end in lines of 64 bytes (8 waves: transposed codes 128), 16 bytes per
// lane.  Several small workgroups on a compute unit are seldom all loading or all storing at once, two large ones often are,
// and a small tensor's waves spread over more units (4 against 8 waves: 50432 x 768 bf16 activation 37 us / 39, 256 x 192
// FP32 with its weight 5.7 / 7.0; two waves 39; the activation takes 31 to 35 today).
// bf16 sources are bound by the vector ALUs, i.e. by the number of instructions.  In us, a 50432 x 3072 bf16 gradient 138 ->
// 129 and activation 117 -> 112: the first two Philox rounds on the scalar unit and once for both streams (SrCounter32), the
// wave's two tiles written out instead of a loop, no cleared destinations for the conversions, one 64-bit address per lane.
// The loop also held 118 registers, now 93: with one stochastic output five waves share a SIMD instead of four (25216 x 384
// activation 13.8 -> 12.0, FP32 gradient 17.3 -> 14.5).  A gradient of bf16
// takes 109 registers for what the streams share; without sharing 95 and 131 us.  FP32 sources are bound by memory
// (50432 x 3072: 170 us, 4.6 TB/s): fetching a second FP32 tile ahead gains 2 % at four waves a SIMD for an activation, and
// spills where both outputs are stochastic (210 us).
// ---------------------------------------------------------------------------
// What a macro tile of 32 * WAVES rows x 128 columns stages in LDS.
template <int WAVES, bool ROWS, bool COLSUM>
struct TileShape {
    static constexpr int THREADS = 64 * WAVES, MACRO_ROWS = 32 * WAVES, MACRO_COLS = 128;
    static constexpr int ROW_PITCH = MACRO_COLS / 2 + 16, COL_PITCH = MACRO_ROWS / 2 + 16;   // bytes per staged line (codes + pad)
    static constexpr int ROW_SCALES = MACRO_COLS / 32, COL_SCALES = MACRO_ROWS / 32;         // scale bytes of a line
    static constexpr int ROW_OFF = 0;                                                        // row codes     [MACRO_ROWS][ROW_PITCH]
    static constexpr int SROW_OFF = ROW_OFF + (ROWS ? MACRO_ROWS * ROW_PITCH : 0);           // row scales    [MACRO_ROWS][ROW_SCALES]
    static constexpr int COL_OFF = SROW_OFF + (ROWS ? MACRO_ROWS * ROW_SCALES : 0);          // transposed    [MACRO_COLS][COL_PITCH]
    static constexpr int SCOL_OFF = COL_OFF + MACRO_COLS * COL_PITCH;                        // their scales  [MACRO_COLS][COL_SCALES]
    static constexpr int CSUM_OFF = SCOL_OFF + MACRO_COLS * COL_SCALES;                      // column sums per wave [WAVES][MACRO_COLS] floats
    static constexpr int BYTES = CSUM_OFF + (COLSUM ? WAVES * MACRO_COLS * 4 : 0);
};

struct TileArgs {
    const void* src;
    const uint8_t* row_codes_in;
    const uint8_t* row_scales_in;
    uint8_t* codes_t;
    uint8_t* scales_t;
    uint8_t* codes_row;
    uint8_t* scales_row;
    int64_t ld;
    uint32_t rows, cols;
    uint32_t src_rows;     // rows the source has; rows from there up to `rows` are zero
    int pre_quant;
    int want_row;          // codes_row is set (an integer: the compiler keeps a pointer's test in a vector register)
    int src_bf16;          // instances for both source types: which one this job reads
    // 1-D grid over macro tiles in row-major order: the first n_wide workgroups own tiles of 128 columns
    // (two 32 x 64 tiles per wave), the rest own the two halves of 64 columns of the tiles after those
    uint32_t n_wide;
    uint32_t wide_per_row; // tiles per block of rows = ceil(cols / 128)
    uint32_t k0, k1, tensor_id_t, tensor_id_row;
    uint64_t index_base;
    const uint32_t* seed_dev;  // when set: the two key words are read from here instead of k0, k1
    float* col_sum_partials;   // COLSUM instances: [ceil(rows / 256)][cols] sums of the source over 256-row blocks, or null
};

// Copies one staged result of a macro tile to memory: `lines` staged lines (rows of row codes, or
// columns of transposed codes), each `pieces` 16-byte pieces of codes (PITCH apart in LDS,
// `code_pitch` bytes apart in memory) and `pieces` scale bytes (SCALES apart in LDS, `scale_pitch` apart
// in memory); pieces <= SCALES.  A lane keeps its piece and steps over the lines, so the loop has no
// index arithmetic beyond two additions; when a line's scale bytes form an aligned 8- or 4-byte
// word they leave as one store.
template <int THREADS, int PITCH, int SCALES>
__device__ __forceinline__ void write_staged(const uint8_t* codes_st, const uint8_t* scales_st,
                                             uint32_t lines, uint32_t pieces,
                                             uint8_t* codes, size_t code_pitch,
                                             uint8_t* scales, size_t scale_pitch, uint32_t tid)
{
    if ((pieces & (pieces - 1u)) == 0u) {
        const uint32_t sh = (uint32_t)__builtin_ctz(pieces);
        const uint32_t lstep = (uint32_t)THREADS >> sh;
        uint32_t l = tid >> sh;
        const uint32_t pc = tid & (pieces - 1u);
        const uint8_t* s = codes_st + l * PITCH + pc * 16;
        uint8_t* d = codes + (size_t)l * code_pitch + pc * 16;
        const size_t dstep = (size_t)lstep * code_pitch;
        for (; l < lines; l += lstep, s += lstep * PITCH, d += dstep)
            *reinterpret_cast<uint4*>(d) = *reinterpret_cast<const uint4*>(s);
    } else {
        for (uint32_t q = tid; q < lines * pieces; q += THREADS) {
            const uint32_t l = q / pieces, pc = q - l * pieces;
            *reinterpret_cast<uint4*>(codes + (size_t)l * code_pitch + pc * 16) =
                *reinterpret_cast<const uint4*>(codes_st + l * PITCH + pc * 16);
        }
    }
    const bool word_ok = ((reinterpret_cast<uintptr_t>(scales) | scale_pitch) & (pieces - 1u)) == 0u;
    if (SCALES == 8 && pieces == 8u && word_ok) {
        for (uint32_t l = tid; l < lines; l += THREADS)
            *reinterpret_cast<uint2*>(scales + (size_t)l * scale_pitch) = *reinterpret_cast<const uint2*>(scales_st + l * SCALES);
    } else if (pieces == 4u && word_ok) {
        for (uint32_t l = tid; l < lines; l += THREADS)
            *reinterpret_cast<uint32_t*>(scales + (size_t)l * scale_pitch) = *reinterpret_cast<const uint32_t*>(scales_st + l * SCALES);
    } else {
        for (uint32_t q = tid; q < lines * SCALES; q += THREADS) {
            const uint32_t l = q / SCALES, pc = q % SCALES;
            if (pc < pieces) scales[(size_t)l * scale_pitch + pc] = scales_st[l * SCALES + pc];
        }
    }
}

// Sums over the 8 lanes that share lane % 8 (the 8 row groups of a wave tile), of the lane's eight columns at once,
// in the fixed order ((g0+g1) + (g2+g3)) + ((g4+g5) + (g6+g7)).  Two values meet in one register at each step: lanes
// whose bit 3 is clear keep the first of a pair, the others the second; then lane-swap instructions pair rows
// of 16 and halves (18 instructions where a reduction per column takes 56).  Returned: the sum of column
// column_of_sum(lane) of the lane's eight.
__device__ __forceinline__ float sum_row_groups8(const float (&v)[8], uint32_t lane)
{
    float p[4];
    const bool second = (lane & 8u) != 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float mine = second ? v[2 * i + 1] : v[2 * i], other = second ? v[2 * i] : v[2 * i + 1];
        p[i] = mine + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(other), 0x128, 0xF, 0xF, true));   // row_ror:8
    }
    float h[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(p[2 * i]), __float_as_uint(p[2 * i + 1]), false, false);
        h[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
    }
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(h[0]), __float_as_uint(h[1]), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}

__device__ __forceinline__ uint32_t column_of_sum(uint32_t lane) { return ((lane >> 3) & 1u) + ((lane >> 4) & 1u) * 2u + (lane >> 5) * 4u; }

// f(0), f(1) with compile-time arguments (the byte a conversion writes is an immediate)
template <typename F>
__device__ __forceinline__ void static_for_pair(F&& f)
{
    f(std::integral_constant<int, 0>{});
    f(std::integral_constant<int, 1>{});
}

// Up to TILE_BATCH_MAX tensors per launch (e.g. the activation and the weight of a layer: one launch,
// and the small tensor's workgroups fill the last round of the large one's).  first[j] is the first
// workgroup of job j (0xFFFFFFFF for unused slots); all jobs share the template parameters.
constexpr int TILE_BATCH_MAX = 4;
struct TileBatch {
    TileArgs job[TILE_BATCH_MAX];
    uint32_t first[TILE_BATCH_MAX];
    mxl::WidenJob widen;   // the grid's last workgroup does this when widen.count is not zero
};

// bf16 -> FP32 of a short vector (a bias, in the launch that quantizes the layer's operands), one workgroup.
__device__ __forceinline__ void widen_bf16(const mxl::WidenJob& j, uint32_t tid, uint32_t threads)
{
    for (uint32_t i = tid; i < j.count; i += threads) j.dst[i] = __uint_as_float((uint32_t)j.src[i] << 16);
}

// SRC: 0 = FP32 source, 1 = bf16 source, 2 = packed row result given
// COLSUM: also the column sums of the source (a bias gradient is that of dY), per 256-row block; a
// separate instance, so that the plain quantizer's code does not change with this feature.
template <typename S, int SRC, bool ROW_SR, bool T_SR, bool FLOOR, bool COLSUM, bool WIDE>
__device__ __forceinline__ void quantize_tile_body(const TileArgs a, const uint32_t block, uint8_t* st)      // a by value: by reference the stochastic
                                                                            // instances take 128 registers and spill
{
    // Philox key: the seed argument, or the 64-bit word in device memory that the caller names (a
    // captured graph then draws new numbers on every replay).  Kept in scalar registers either way.
    uint32_t k0 = a.k0, k1 = a.k1;
    if ((ROW_SR || T_SR) && a.seed_dev) {
        k0 = __builtin_amdgcn_readfirstlane(a.seed_dev[0]);
        k1 = __builtin_amdgcn_readfirstlane(a.seed_dev[1]);
    }
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int cc = lane & 7, rg = lane >> 3;
    const int wr = wave;                                  // wave position inside the macro tile
    // macro tile of this workgroup (uniform): a wide one, or one half of a wide one
    const bool wide = block < a.n_wide;
    const uint32_t narrow = wide ? 0u : block - a.n_wide;
    // Workgroup ids go round the 8 XCDs, each with its own L2.  A macro tile writes 4 scale bytes per row
    // and 8 per column: a 32-byte sector of a scale array is completed by up to 8 tiles side by side, or 4
    // on top of each other.  Each XCD therefore takes a contiguous range of the row-major tile order, so
    // that the tiles which share sectors meet in one L2 and the sectors leave it whole.
    const uint32_t xcd_class = block & 7u, per_xcd = a.n_wide >> 3, rem_xcd = a.n_wide & 7u;
    const uint32_t wide_index = wide ? xcd_class * per_xcd + min(xcd_class, rem_xcd) + (block >> 3)
                                     : a.n_wide + (narrow >> 1);
    const uint32_t row_block = wide_index / a.wide_per_row;
    const int tiles_per_wave = wide ? 2 : 1;
    const uint32_t macro_rows = S::MACRO_ROWS, macro_cols = 64u * tiles_per_wave;
    const uint32_t mrow0 = row_block * macro_rows;        // macro tile origin
    const uint32_t mcol0 = (wide_index - row_block * a.wide_per_row) * 128u + (wide ? 0u : (narrow & 1u) * 64u);
    if (mcol0 >= a.cols) return;                          // second half of a tile that is only 64 columns wide
    const bool wave_has_rows = mrow0 + wr * 32 < a.rows;
    const bool wave_rows_full = mrow0 + wr * 32 + 32 <= a.src_rows;
    const uint32_t lrow0 = wr * 32 + 4 * rg;              // first of this lane's 4 rows inside the macro tile
    const uint32_t row0 = mrow0 + lrow0;
    const bool want_row = SRC != 2 && a.want_row;
    const uint32_t half_rows = a.rows >> 1, grp_rows = a.rows >> 5;
    const uint32_t half_cols = a.cols >> 1, grp_cols = a.cols >> 5;

    // Element (row0 + j, c + t) has index index_base + (row0 + j) * cols + c + t: one Philox block of 8 per row.
    using Blk = std::conditional_t<WIDE, uint64_t, uint32_t>;
    const uint32_t blk_row = a.cols >> 3, blk_hi = (uint32_t)(a.index_base >> 35);
    const Blk blk0 = (Blk)(a.index_base >> 3) + (Blk)row0 * blk_row + (mcol0 >> 3) + cc;

    // A lane's four rows of 8 elements, as loaded: bf16 values stay packed in pairs, packed results stay codes.
    // The second tile's are fetched while the first one is encoded.
    using Row = Raw8<std::conditional_t<SRC == 0, float, uint16_t>>;
    struct Tile {
        Row x[SRC == 2 ? 1 : 4];
        uint32_t pk[SRC == 2 ? 4 : 1], byte[SRC == 2 ? 4 : 1];
    };
    // the lane's first element; the rows and the second tile are uniform offsets from it
    using SrcT = std::conditional_t<SRC == 0, float, uint16_t>;
    const SrcT* lane_src = nullptr;
    const uint8_t *lane_codes = nullptr, *lane_scales = nullptr;
    if constexpr (SRC == 2) {
        lane_codes = a.row_codes_in + ((size_t)(mrow0 + wr * 32) * half_cols + (mcol0 >> 1)) + ((uint64_t)(uint32_t)(4 * rg) * half_cols + (uint32_t)(cc * 4));
        lane_scales = a.row_scales_in + ((size_t)(mrow0 + wr * 32) * grp_cols + (mcol0 >> 5)) + ((uint64_t)(uint32_t)(4 * rg) * grp_cols + (uint32_t)(cc >> 2));
    } else
        lane_src = static_cast<const SrcT*>(a.src) + ((int64_t)(mrow0 + wr * 32) * a.ld + mcol0) + ((uint64_t)(uint32_t)(4 * rg) * (uint64_t)a.ld + (uint32_t)(cc * 8));
    auto load_row = [&](Row& r, int j, int ci) {
        const SrcT* p = lane_src + j * a.ld + ci * 64;
        if constexpr (SRC == 0)      r = load8(p);
        else if constexpr (SRC == 1) r = load8_raw(p);
    };
    auto fetch = [&](Tile& d, int ci) {
        const uint32_t col = mcol0 + ci * 64 + cc * 8;
        if constexpr (SRC == 2) {
            const uint8_t *pc = lane_codes + ci * 32, *ps = lane_scales + ci * 2;
            if (mcol0 + ci * 64 + 64 <= a.cols) {                              // uniform: no masking
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    d.pk[j] = *reinterpret_cast<const uint32_t*>(pc + (size_t)j * half_cols);
                    d.byte[j] = ps[(size_t)j * grp_cols];
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    d.pk[j] = 0u; d.byte[j] = 98u;
                    if (col < a.cols) {
                        d.pk[j] = *reinterpret_cast<const uint32_t*>(pc + (size_t)j * half_cols);
                        d.byte[j] = ps[(size_t)j * grp_cols];
                    }
                }
            }
        } else if (wave_rows_full && mcol0 + ci * 64 + 64 <= a.cols) {       // uniform: no masking
#pragma unroll
            for (int j = 0; j < 4; ++j) load_row(d.x[j], j, ci);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if constexpr (SRC == 0) d.x[j] = zero8();
                else                    d.x[j] = bf16x8_raw{0u, 0u, 0u, 0u};
                if (col < a.cols && row0 + j < a.src_rows) load_row(d.x[j], j, ci);
            }
        }
    };
    auto element = [](const Row& r, int t) -> float { return element_of(r, t); };

    constexpr bool PREFETCH = SRC != 0 || (!ROW_SR && T_SR);   // FP32: 32 registers for the second tile
    auto encode = [&](const Tile& cur, auto ci_c) {
        constexpr int ci = decltype(ci_c)::value;
        const uint32_t lcol0 = ci * 64 + cc * 8;          // first of this lane's 8 columns inside the macro tile
        // ---- column sums of the source over this wave's 32 rows -------------
        if (COLSUM && SRC != 2 && a.col_sum_partials != nullptr) {
            f32_round_to_nearest_even();
            float cs[8];
            Row x[4] = {cur.x[0], cur.x[1], cur.x[2], cur.x[3]};
            if constexpr (SRC == 1) {
                // opaque copies: the values unpacked here are not kept (32 registers) for the phases below
#pragma unroll
                for (int j = 0; j < 4; ++j) asm("" : "+v"(x[j]));
            }
#pragma unroll
            for (int t = 0; t < 8; ++t)
                cs[t] = ((element(x[0], t) + element(x[1], t)) + element(x[2], t)) + element(x[3], t);
            reinterpret_cast<float*>(st + S::CSUM_OFF)[wr * 128 + lcol0 + column_of_sum(lane)] = sum_row_groups8(cs, lane);
            __builtin_amdgcn_sched_barrier(0);            // the random numbers of later phases stay out of this one's registers
        }
        // ---- bf16: group maxima, scale bytes of two rows per register ----
        // The magnitudes serve the row maxima and, where the column groups take the source itself, the column maxima.
        const bool rows_wanted = want_row || a.pre_quant;
        uint32_t rbytes[2], cmax[4];
        if constexpr (SRC == 1) {
            auto maxima = [&](auto rows_c, auto cols_c) {
                uint32_t rm[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    uint32_t k[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) k[i] = cur.x[j][i] & 0x7FFF7FFFu;
                    if constexpr (rows_c.value) rm[j] = pk_max(pk_max(k[0], k[1]), pk_max(k[2], k[3]));
                    if constexpr (cols_c.value) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) cmax[i] = j ? pk_max(cmax[i], k[i]) : k[i];
                    }
                }
                if constexpr (rows_c.value) {
                    rbytes[0] = scale_bytes_bf16<FLOOR>(quad_amax_bf16_rows(rm[0], rm[1]));
                    rbytes[1] = scale_bytes_bf16<FLOOR>(quad_amax_bf16_rows(rm[2], rm[3]));
                }
            };
            if (a.pre_quant)   maxima(std::true_type{}, std::false_type{});
            else if (want_row) maxima(std::true_type{}, std::true_type{});
            else               maxima(std::false_type{}, std::true_type{});
        }
        // ---- random numbers: what both streams have in common is made once ----
        constexpr bool SHARE = ROW_SR && T_SR && (SRC == 1 || COLSUM);     // FP32 gradients: five waves a SIMD are worth more
        auto counter = [&](int j) { return sr_counter(blk0 + (Blk)(ci * 8) + (Blk)j * blk_row, k1); };
        decltype(counter(0)) shared[4];
        if constexpr (SHARE) {
#pragma unroll
            for (int j = 0; j < 4; ++j) shared[j] = counter(j);
        }
        auto counter_of = [&](int j) {
            if constexpr (SHARE) return shared[j];
            else                 return counter(j);
        };
        // ---- 1x32 quantizer: codes of the lane's four rows and their scales ----
        uint32_t pk[4];
        float row_scale[4];
        if constexpr (SRC == 2) {
#pragma unroll
            for (int j = 0; j < 4; ++j) { pk[j] = cur.pk[j]; row_scale[j] = scale_operand(cur.byte[j]); }
        } else if (rows_wanted) {
            if (ROW_SR) f32_round_toward_plus_inf();
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint32_t byte;
                if constexpr (SRC == 0) byte = row_scale_byte<FLOOR>(cur.x[j]);
                else                    byte = (j & 1) ? rbytes[j >> 1] >> 16 : rbytes[j >> 1] & 0xFFFFu;
                row_scale[j] = scale_operand(byte);
                if constexpr (ROW_SR)
                    pk[j] = sr_codes8<FLOOR>(cur.x[j], byte, sr_terms(counter_of(j), blk_hi, a.tensor_id_row, k0, k1));
                else
                    pk[j] = rtn_codes8(cur.x[j], byte);
                if (want_row) {
                    *reinterpret_cast<uint32_t*>(st + S::ROW_OFF + (lrow0 + j) * S::ROW_PITCH + (lcol0 >> 1)) = pk[j];
                    if ((cc & 3) == 0) st[S::SROW_OFF + (lrow0 + j) * S::ROW_SCALES + (lcol0 >> 5)] = (uint8_t)byte;
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // ---- 32x1 quantizer: group = this lane's 4 rows x the 8 lanes sharing cc ----
        // Scale bytes of the lane's eight columns, two per register: byte_of(t).
        uint32_t sb[4];
        auto column_byte = [&](int t) { return (t & 1) ? sb[t >> 1] >> 16 : sb[t >> 1] & 0xFFFFu; };      // (FP32 sources: see there)
        auto store_column_bytes = [&](uint32_t two, uint32_t first, uint32_t step) {
            // rows of 16 lanes 0..3 hold the columns first + step * {0, 2, 1, 3}: the lanes of each row's first half write
            if ((lane & 8) == 0) {
                st[S::SCOL_OFF + (lcol0 + first) * S::COL_SCALES + wr] = (uint8_t)two;
                st[S::SCOL_OFF + (lcol0 + first + step) * S::COL_SCALES + wr] = (uint8_t)(two >> 16);
            }
        };
        const uint32_t row16 = (uint32_t)lane >> 4, place = ((row16 & 1u) << 1) | (row16 >> 1);
        auto column_bytes_bf16 = [&](const uint32_t (&m)[4]) {
            const uint32_t two = scale_bytes_bf16<FLOOR>(reduce_row_groups4(m, [](uint32_t p, uint32_t q) { return pk_max(p, q); }));
            store_column_bytes(two, 2u * place, 1u);
            spread_row_groups4(two, sb);
        };
        uint32_t colpk[8];                                // the lower 16 bits are written and stored
        auto terms = [&](int j) { return sr_terms(counter_of(j), blk_hi, a.tensor_id_t, k0, k1); };
        if (SRC == 2 || a.pre_quant) {
            uint32_t m[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t mags = pk[j] & 0x77777777u;
                m[0] = pk_max(m[0], cvt_bf16_fp4<0>(mags, row_scale[j]));
                m[1] = pk_max(m[1], cvt_bf16_fp4<1>(mags, row_scale[j]));
                m[2] = pk_max(m[2], cvt_bf16_fp4<2>(mags, row_scale[j]));
                m[3] = pk_max(m[3], cvt_bf16_fp4<3>(mags, row_scale[j]));
            }
            column_bytes_bf16(m);
            // Uniform and rare (the scale operand of byte 0 is zero).  With the mask on every element instead, 50432 x 3072 from
            // packed codes takes 70.9 us against 67.4.
            const bool any_byte_0 = T_SR && __any(__builtin_fminf(__builtin_fminf(row_scale[0], row_scale[1]), __builtin_fminf(row_scale[2], row_scale[3])) == 0.0f);
            if (T_SR) f32_round_toward_plus_inf();
            static_for_pair([&](auto jp_c) {
                constexpr int jp = decltype(jp_c)::value;
                float d[2][8];                            // T_SR: on the grid; otherwise the dequantized values
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int j = 2 * jp + r;
                    U8 rnd;
                    if (T_SR) rnd = terms(j);
                    const f32x2_hw v[4] = {cvt_f32_fp4<0>(pk[j], row_scale[j]), cvt_f32_fp4<1>(pk[j], row_scale[j]),
                                           cvt_f32_fp4<2>(pk[j], row_scale[j]), cvt_f32_fp4<3>(pk[j], row_scale[j])};
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        d[r][t] = v[t >> 1][t & 1];
                        if (T_SR) d[r][t] = __uint_as_float(sr_grid_dequantized<FLOOR>(d[r][t], 1 - (int)column_byte(t), rnd.w[t]));
                    }
                }
                if (T_SR && any_byte_0) {
#pragma unroll
                    for (int r = 0; r < 2; ++r)
#pragma unroll
                        for (int t = 0; t < 8; ++t) d[r][t] = __uint_as_float(__float_as_uint(d[r][t]) & ON_GRID);
                }
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    if constexpr (T_SR)         colpk[t] = pack_grid<jp>(jp ? colpk[t] : __float_as_uint(d[0][t]), __float_as_uint(d[0][t]), __float_as_uint(d[1][t]));
                    else if constexpr (jp == 0) colpk[t] = cvt_rtn_f32<0>(d[0][t], d[1][t], scale_operand(column_byte(t)));
                    else                        colpk[t] = cvt_rtn_f32<1>(colpk[t], d[0][t], d[1][t], scale_operand(column_byte(t)));
                }
            });
        } else if constexpr (SRC == 1) {
            column_bytes_bf16(cmax);
            if (T_SR) f32_round_toward_plus_inf();
            static_for_pair([&](auto jp_c) {
                constexpr int jp = decltype(jp_c)::value;
                if constexpr (T_SR) {
                    uint32_t g[2][8];
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        const U8 rnd = terms(2 * jp + r);
#pragma unroll
                        for (int t = 0; t < 8; ++t) {
                            g[r][t] = sr_grid<FLOOR>(element(cur.x[2 * jp + r], t), 1 - (int)column_byte(t), rnd.w[t]);
                        }
                    }
#pragma unroll
                    for (int t = 0; t < 8; ++t) colpk[t] = pack_grid<jp>(jp ? colpk[t] : g[0][t], g[0][t], g[1][t]);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t n0 = ties_to_larger(cur.x[2 * jp][i]), n1 = ties_to_larger(cur.x[2 * jp + 1][i]);
                        // the two rows of one column side by side
                        const uint32_t lo = __builtin_amdgcn_perm(n1, n0, 0x05040100u), hi = __builtin_amdgcn_perm(n1, n0, 0x07060302u);
                        colpk[2 * i] = cvt_fp4_bf16<jp>(jp ? colpk[2 * i] : lo, lo, scale_operand(sb[i] & 0xFFFFu));
                        colpk[2 * i + 1] = cvt_fp4_bf16<jp>(jp ? colpk[2 * i + 1] : hi, hi, scale_operand(sb[i] >> 16));
                    }
                }
            });
        } else if constexpr (SRC == 0) {
            // FP32 maxima: eight values, reduced four at a time and packed as bytes: registers hold columns (i, i + 4)
            uint32_t lo[4], hi[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                lo[i] = absmax3_bits(cur.x[2].v[i], cur.x[3].v[i], absmax3_bits(cur.x[0].v[i], cur.x[1].v[i], 0u));
                hi[i] = absmax3_bits(cur.x[2].v[i + 4], cur.x[3].v[i + 4], absmax3_bits(cur.x[0].v[i + 4], cur.x[1].v[i + 4], 0u));
            }
            auto umax = [](uint32_t p, uint32_t q) { return p > q ? p : q; };
            const uint32_t two = scale_byte(reduce_row_groups4(lo, umax), FLOOR) | scale_byte(reduce_row_groups4(hi, umax), FLOOR) << 16;
            store_column_bytes(two, place, 4u);
            spread_row_groups4(two, sb);
            if (T_SR) f32_round_toward_plus_inf();
            static_for_pair([&](auto jp_c) {
                constexpr int jp = decltype(jp_c)::value;
                auto byte_f32 = [&](int t) { return t >= 4 ? sb[t & 3] >> 16 : sb[t & 3] & 0xFFFFu; };
                if constexpr (T_SR) {
                    uint32_t g[2][8];
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        const U8 rnd = terms(2 * jp + r);
#pragma unroll
                        for (int t = 0; t < 8; ++t) g[r][t] = sr_grid<FLOOR>(cur.x[2 * jp + r].v[t], 1 - (int)byte_f32(t), rnd.w[t]);
                    }
#pragma unroll
                    for (int t = 0; t < 8; ++t) colpk[t] = pack_grid<jp>(jp ? colpk[t] : g[0][t], g[0][t], g[1][t]);
                } else {
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        if constexpr (jp == 0) colpk[t] = cvt_rtn_f32<0>(cur.x[0].v[t], cur.x[1].v[t], scale_operand(byte_f32(t)));
                        else                   colpk[t] = cvt_rtn_f32<1>(colpk[t], cur.x[2].v[t], cur.x[3].v[t], scale_operand(byte_f32(t)));
                    }
                }
            });
        }
#pragma unroll
        for (int t = 0; t < 8; ++t)
            *reinterpret_cast<uint16_t*>(st + S::COL_OFF + (lcol0 + t) * S::COL_PITCH + (lrow0 >> 1)) = (uint16_t)colpk[t];
    };
    // Written out twice and not a loop: handing the fetched registers on costs 14 moves a tile.
    if (wave_has_rows) {
        const bool second = wide && mcol0 + 64 < a.cols;  // uniform
        Tile t0, t1;
        fetch(t0, 0);
        if (PREFETCH && second) fetch(t1, 1);
        encode(t0, std::integral_constant<int, 0>{});
        __builtin_amdgcn_sched_barrier(0);
        if (second) {
            if (!PREFETCH) fetch(t1, 1);
            encode(t1, std::integral_constant<int, 1>{});
        }
    }
    __syncthreads();

    // ---- write the staged macro tile out: 16 bytes per lane, whole 128-byte lines ----
    const uint32_t ncols_here = min(macro_cols, a.cols - mcol0);    // multiples of 32
    const uint32_t nrows_here = min(macro_rows, a.rows - mrow0);    // multiples of 32
    if (want_row)
        write_staged<S::THREADS, S::ROW_PITCH, S::ROW_SCALES>(st + S::ROW_OFF, st + S::SROW_OFF, nrows_here, ncols_here >> 5,
                     a.codes_row + (size_t)mrow0 * half_cols + (mcol0 >> 1), half_cols,
                     a.scales_row + (size_t)mrow0 * grp_cols + (mcol0 >> 5), grp_cols, tid);
    write_staged<S::THREADS, S::COL_PITCH, S::COL_SCALES>(st + S::COL_OFF, st + S::SCOL_OFF, ncols_here, nrows_here >> 5,
                 a.codes_t + (size_t)mcol0 * half_rows + (mrow0 >> 1), half_rows,
                 a.scales_t + (size_t)mcol0 * grp_rows + (mrow0 >> 5), grp_rows, tid);
    if (COLSUM && a.col_sum_partials != nullptr && (uint32_t)tid < ncols_here) {
        // the waves that had rows, in order; one value per column of this 256-row block.  Round to
        // nearest like the per-wave sums (no quantizer arithmetic follows, the mode is not restored).
        f32_round_to_nearest_even();
        const float* cs = reinterpret_cast<const float*>(st + S::CSUM_OFF) + tid;
        float s = cs[0];
        for (uint32_t w = 1; w < (nrows_here >> 5); ++w) s += cs[w * 128];
        a.col_sum_partials[(size_t)row_block * a.cols + mcol0 + tid] = s;
    }
}

// Waves of a launch that share a SIMD, as the registers of its instance allow (the kernels' launch bounds say so too).
// src: 0 FP32, 1 bf16, 2 packed codes.  Eight-wave workgroups: two on a compute unit (the registers of an instance without
// stochastic columns would do for three).
constexpr int tile_waves_per_simd(int src, bool row_sr, bool t_sr, int waves)
{
    if (waves == 8) return 4;
    if (src == 2) return 8;
    if (!t_sr) return src == 1 || row_sr ? 6 : 5;
    if (src == 1) return row_sr ? 4 : 5;
    return row_sr ? 5 : 4;
}

// SRC as above, or 3: FP32 and bf16 jobs in one launch (a bf16 activation and its FP32 master weight).
// WIDE: block numbers of the launch differ in their upper word (SrCounter64).
template <int SRC, bool ROW_SR, bool T_SR, bool FLOOR, bool COLSUM, int WAVES, bool WIDE>
__global__ __launch_bounds__(64 * WAVES, tile_waves_per_simd(SRC == 3 ? 0 : SRC, ROW_SR, T_SR, WAVES)) void quantize_tile_kernel(TileBatch batch)
{
    using S = TileShape<WAVES, SRC != 2, COLSUM>;
    __shared__ __attribute__((aligned(16))) uint8_t st[S::BYTES];
    if (batch.widen.count != 0u && blockIdx.x == gridDim.x - 1u) {
        widen_bf16(batch.widen, threadIdx.x, S::THREADS);
        return;
    }
    uint32_t job = 0;
#pragma unroll
    for (int i = 1; i < TILE_BATCH_MAX; ++i) job += blockIdx.x >= batch.first[i] ? 1u : 0u;
    const TileArgs a = batch.job[job];
    const uint32_t block = blockIdx.x - batch.first[job];
    if constexpr (SRC == 3) {
        if (a.src_bf16) quantize_tile_body<S, 1, ROW_SR, T_SR, FLOOR, COLSUM, WIDE>(a, block, st);
        else            quantize_tile_body<S, 0, ROW_SR, T_SR, FLOOR, COLSUM, WIDE>(a, block, st);
    } else {
        quantize_tile_body<S, SRC, ROW_SR, T_SR, FLOOR, COLSUM, WIDE>(a, block, st);
    }
}

// (the order is fixed: see mx_device.hpp)
__global__ __launch_bounds__(256) void column_sum_finish_kernel(mxl::ColumnSumTail t)
{
    mxl::column_sum_finish(t, blockIdx.x);
}

// ---------------------------------------------------------------------------
// Q-Ramping's oscillation detection (Sec. 6.1): one step of
//     dist_W += |w - w_prev|,   dist_Q += |w_Q - w_Q,prev|,   w_Q = P * 2^s,
// per weight element, FP32, one rounding per operation.  The previous quantized weight is kept
// packed (codes_prev / scales_prev), not as FP32: 0.53 instead of 4 bytes per element of state.
// One lane owns 8 consecutive elements, as in the quantizers.
// ---------------------------------------------------------------------------
struct OscArgs {
    const void* w;
    const uint8_t* codes;
    const uint8_t* scales;
    float* w_prev;
    uint8_t* codes_prev;
    uint8_t* scales_prev;
    float* dist_w;
    float* dist_q;
    int64_t ld;
    uint32_t cpr;          // 8-element chunks per row
    uint32_t total;        // rows * cpr
    int init;
};

template <typename SrcT>
__global__ __launch_bounds__(ROWS_THREADS) void oscillation_kernel(OscArgs a)
{
    const uint32_t q = blockIdx.x * ROWS_THREADS + threadIdx.x;
    if (q >= a.total) return;
    const uint32_t r = q / a.cpr, ch = q - r * a.cpr;
    const F8 w = load8(static_cast<const SrcT*>(a.w) + (int64_t)r * a.ld + (int64_t)ch * 8);
    const size_t dense = (size_t)q * 8;                   // state arrays are dense [rows][cols]
    const uint32_t pk = reinterpret_cast<const uint32_t*>(a.codes)[q];
    const uint32_t byte = a.scales[(size_t)q >> 2];       // cols/32 groups per row = cpr/4
    float4* wp = reinterpret_cast<float4*>(a.w_prev + dense);
    if (!a.init) {
        const uint32_t pk0 = reinterpret_cast<const uint32_t*>(a.codes_prev)[q];
        const uint32_t byte0 = a.scales_prev[(size_t)q >> 2];
        const float4 p0 = wp[0], p1 = wp[1];
        const float prev[8] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w};
        float4* dwp = reinterpret_cast<float4*>(a.dist_w + dense);
        float4* dqp = reinterpret_cast<float4*>(a.dist_q + dense);
        const float4 a0 = dwp[0], a1 = dwp[1], b0 = dqp[0], b1 = dqp[1];
        float dw[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
        float dq[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const float wq = dequant((pk >> (4 * t)) & 15u, byte);
            const float wq0 = dequant((pk0 >> (4 * t)) & 15u, byte0);
            dw[t] = __fadd_rn(dw[t], __builtin_fabsf(__fsub_rn(w.v[t], prev[t])));
            dq[t] = __fadd_rn(dq[t], __builtin_fabsf(__fsub_rn(wq, wq0)));
        }
        dwp[0] = make_float4(dw[0], dw[1], dw[2], dw[3]);
        dwp[1] = make_float4(dw[4], dw[5], dw[6], dw[7]);
        dqp[0] = make_float4(dq[0], dq[1], dq[2], dq[3]);
        dqp[1] = make_float4(dq[4], dq[5], dq[6], dq[7]);
    } else {
        const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
        reinterpret_cast<float4*>(a.dist_w + dense)[0] = z;
        reinterpret_cast<float4*>(a.dist_w + dense)[1] = z;
        reinterpret_cast<float4*>(a.dist_q + dense)[0] = z;
        reinterpret_cast<float4*>(a.dist_q + dense)[1] = z;
    }
    wp[0] = make_float4(w.v[0], w.v[1], w.v[2], w.v[3]);
    wp[1] = make_float4(w.v[4], w.v[5], w.v[6], w.v[7]);
    reinterpret_cast<uint32_t*>(a.codes_prev)[q] = pk;
    if ((ch & 3) == 0) a.scales_prev[(size_t)q >> 2] = (uint8_t)byte;
}

// Amplification factor of Algorithm 2 (Q-Ramping): N_w = min(k2 * floor(R_w / k1) + 1, n_max),
// R_w = dist_Q / dist_W with IEEE FP32 divisions; dist_W = 0 gives R_w = 0 if dist_Q = 0, else +inf.
__global__ void ramping_factor_kernel(const float* dist_w, const float* dist_q, int64_t count,
                                      float k1, int k2, int n_max, int32_t* factor)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const float dw = dist_w[i], dq = dist_q[i];
    float ratio;
    if (dw == 0.0f) ratio = dq == 0.0f ? 0.0f : __builtin_inff();
    else            ratio = __fdiv_rn(dq, dw);
    const float steps = floorf(__fdiv_rn(ratio, k1));
    int32_t n = n_max;
    if (steps < (float)n_max) {
        const int64_t v = (int64_t)k2 * (int64_t)steps + 1;
        n = v < (int64_t)n_max ? (int32_t)v : n_max;
    }
    factor[i] = n;
}

// ---------------------------------------------------------------------------
// Quantization confidence (Sec. 4.2) on the latent value y = w / S of a 1x32 group:
//     conf = min_i |y - thrd_i| / MaxDist(y_FP4).
// The thresholds are the midpoints of neighbouring E2M1 values; the cell of an E2M1 value reaches
// from the threshold below to the threshold above it (the cell of 0 is [-0.25, 0.25], the cell of
// 6 is [5, 6]), and MaxDist is half the cell's width, for the outermost cell the whole width.
// The sign plays no part: everything is taken on a = |y|.  y is exact (a power-of-two scaling),
// each distance is one FP32 subtraction, the quotient one IEEE division.
// ---------------------------------------------------------------------------
struct ConfArgs {
    const void* w;
    float* conf;                       // may be null
    unsigned long long* hist;          // may be null
    int64_t ld;
    uint32_t cpr, total;
    int bins;
    int floor_mode;
};

__device__ __forceinline__ float confidence_of(float a)
{
    // lower threshold, upper threshold, MaxDist of the cell that holds a
    float lo, hi, den;
    if (a < 0.25f)      { lo = -0.25f; hi = 0.25f; den = 0.25f; }
    else if (a < 0.75f) { lo = 0.25f;  hi = 0.75f; den = 0.25f; }
    else if (a < 1.25f) { lo = 0.75f;  hi = 1.25f; den = 0.25f; }
    else if (a < 1.75f) { lo = 1.25f;  hi = 1.75f; den = 0.25f; }
    else if (a < 2.5f)  { lo = 1.75f;  hi = 2.5f;  den = 0.375f; }
    else if (a < 3.5f)  { lo = 2.5f;   hi = 3.5f;  den = 0.5f; }
    else if (a < 5.0f)  { lo = 3.5f;   hi = 5.0f;  den = 0.75f; }
    else                { lo = 5.0f;   hi = __builtin_inff(); den = 1.0f; }
    const float below = __fsub_rn(a, lo), above = __fsub_rn(hi, a);
    return __fdiv_rn(below < above ? below : above, den);
}

constexpr int CONF_MAX_BINS = mxl::CONFIDENCE_MAX_BINS;

template <typename SrcT>
__global__ __launch_bounds__(ROWS_THREADS) void confidence_kernel(ConfArgs a)
{
    __shared__ uint32_t lh[CONF_MAX_BINS];
    if (a.hist) {
        for (int b = threadIdx.x; b < a.bins; b += ROWS_THREADS) lh[b] = 0u;
        __syncthreads();
    }
    // a.total is a multiple of 4 and a quad of lanes (one 1x32 group) starts at a multiple of 4:
    // the lanes of a group pass or fail the loop test together
    for (uint32_t q = blockIdx.x * ROWS_THREADS + threadIdx.x; q < a.total; q += gridDim.x * ROWS_THREADS) {
        const uint32_t r = q / a.cpr, ch = q - r * a.cpr;
        const F8 w = load8(static_cast<const SrcT*>(a.w) + (int64_t)r * a.ld + (int64_t)ch * 8);
        const uint32_t byte = scale_byte(quad_max(amax_bits8(w)), a.floor_mode);
        const float inv = inv_scale(byte);
        float c[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            float y = __builtin_fabsf(__fmul_rn(w.v[t], inv));
            y = y > 6.0f ? 6.0f : y;                       // Eq. 2's scale truncates to Q_p
            c[t] = confidence_of(y);
        }
        if (a.conf) {
            float4* out = reinterpret_cast<float4*>(a.conf + (size_t)q * 8);
            out[0] = make_float4(c[0], c[1], c[2], c[3]);
            out[1] = make_float4(c[4], c[5], c[6], c[7]);
        }
        if (a.hist) {
            const float nb = (float)a.bins;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                int b = (int)floorf(__fmul_rn(c[t], nb));
                b = b > a.bins - 1 ? a.bins - 1 : b;
                atomicAdd(&lh[b], 1u);
            }
        }
    }
    if (a.hist) {
        __syncthreads();
        for (int b = threadIdx.x; b < a.bins; b += ROWS_THREADS)
            if (lh[b]) atomicAdd(&a.hist[b], (unsigned long long)lh[b]);
    }
}

// ---------------------------------------------------------------------------
// One term of the rate of change (Sec. 4.1): ||x - x_prev||_F / ||x_prev||_F, then x_prev = x.
// Differences of FP32 values and their squares' sums are taken in FP64.  The order of the sums is
// fixed by the launch shape (RATE_BLOCKS x ROWS_THREADS lanes, grid-stride over 8-element chunks,
// then a tree within the block, then the blocks in index order), so a call repeats bit for bit.
// ---------------------------------------------------------------------------
constexpr int RATE_BLOCKS = 1024;

struct RateArgs {
    const void* x;
    float* x_prev;
    double* partial;                   // [RATE_BLOCKS][2]
    int64_t ld;
    uint32_t cpr, total;
    int init;
};

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    return v;
}

template <typename SrcT>
__global__ __launch_bounds__(ROWS_THREADS) void rate_partial_kernel(RateArgs a)
{
    __shared__ double red[2][ROWS_THREADS / 64];
    double diff2 = 0.0, prev2 = 0.0;
    for (uint32_t q = blockIdx.x * ROWS_THREADS + threadIdx.x; q < a.total; q += RATE_BLOCKS * ROWS_THREADS) {
        const uint32_t r = q / a.cpr, ch = q - r * a.cpr;
        const F8 x = load8(static_cast<const SrcT*>(a.x) + (int64_t)r * a.ld + (int64_t)ch * 8);
        float4* pp = reinterpret_cast<float4*>(a.x_prev + (size_t)q * 8);
        if (!a.init) {
            const float4 p0 = pp[0], p1 = pp[1];
            const float old[8] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w};
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const double o = (double)old[t], d = (double)x.v[t] - o;
                diff2 = fma(d, d, diff2);
                prev2 = fma(o, o, prev2);
            }
        }
        pp[0] = make_float4(x.v[0], x.v[1], x.v[2], x.v[3]);
        pp[1] = make_float4(x.v[4], x.v[5], x.v[6], x.v[7]);
    }
    diff2 = wave_sum(diff2);
    prev2 = wave_sum(prev2);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) { red[0][wave] = diff2; red[1][wave] = prev2; }
    __syncthreads();
    if (threadIdx.x == 0) {
        double d = 0.0, p = 0.0;
        for (int i = 0; i < ROWS_THREADS / 64; ++i) { d += red[0][i]; p += red[1][i]; }
        a.partial[2 * blockIdx.x] = d;
        a.partial[2 * blockIdx.x + 1] = p;
    }
}

// result[0] = this step's term, result[1] = sum of the terms since the window opened,
// result[2] = their number.  One workgroup.
__global__ __launch_bounds__(ROWS_THREADS) void rate_finish_kernel(const double* partial, int init, double* result)
{
    __shared__ double red[2][ROWS_THREADS / 64];
    double d = 0.0, p = 0.0;
    for (int b = threadIdx.x; b < RATE_BLOCKS; b += ROWS_THREADS) { d += partial[2 * b]; p += partial[2 * b + 1]; }
    d = wave_sum(d);
    p = wave_sum(p);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) { red[0][wave] = d; red[1][wave] = p; }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (init) {
            result[0] = 0.0; result[1] = 0.0; result[2] = 0.0;
        } else {
            double dd = 0.0, pp = 0.0;
            for (int i = 0; i < ROWS_THREADS / 64; ++i) { dd += red[0][i]; pp += red[1][i]; }
            double term;
            if (pp == 0.0) term = dd == 0.0 ? 0.0 : (double)__builtin_inff();
            else           term = sqrt(dd) / sqrt(pp);
            result[0] = term;
            result[1] = result[1] + term;
            result[2] = result[2] + 1.0;
        }
    }
}

__global__ void dequantize_kernel(const uint8_t* codes, const uint8_t* scales, int64_t total_bytes,
                                  int64_t cols, float* out)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;     // one code byte = 2 elements
    if (i >= total_bytes) return;
    int64_t half = cols >> 1;
    int64_t r = i / half, j = i - r * half;
    uint32_t byte = scales[r * (cols >> 5) + (j >> 4)];
    uint32_t b = codes[i];
    out[2 * i] = dequant(b & 15u, byte);
    out[2 * i + 1] = dequant(b >> 4, byte);
}

__global__ void dequantize_e3m0_kernel(const uint8_t* codes, const uint8_t* scales, int64_t total, int64_t cols, float* out)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;       // index of a code byte
    if (i >= total) return;
    int64_t half = cols >> 1;
    int64_t r = i / half, j = i - r * half;
    uint32_t byte = scales[r * (cols >> 5) + (j >> 4)];
    uint32_t b = codes[i];
    out[2 * i] = dequant_e3m0(b & 15u, byte);
    out[2 * i + 1] = dequant_e3m0(b >> 4, byte);
}

__global__ __launch_bounds__(256) void calibration_copy_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) dst[i] = src[i];
}

}  // namespace

// ------------------------------------------------------------------ launchers

namespace mxl {

// Whether the Philox block numbers of elements [index_base, index_base + 8 * blocks) differ in their upper 32 bits.  Those
// of a tensor of fewer than 2^35 elements without an index base never do; the others run the kernels' WIDE instances.
static bool spans_counter_words(uint64_t index_base, uint64_t blocks)
{
    const uint64_t first = index_base >> 3;
    return (first >> 32) != ((first + blocks - 1) >> 32);
}

hipError_t launch_quantize_rows(const QuantRowsParams& p, hipStream_t st)
{
    RowsArgs a{};
    a.src = p.src; a.codes = p.codes; a.scales = p.scales; a.ema = nullptr;
    a.ld = p.ld; a.cpr = (uint32_t)(p.cols / 8); a.total = (uint32_t)(p.rows * (p.cols / 8));
    a.contiguous = p.ld == p.cols; a.floor_mode = p.floor_mode;
    a.k0 = (uint32_t)p.seed; a.k1 = (uint32_t)(p.seed >> 32); a.tensor_id = p.tensor_id;
    a.base_blk = p.index_base >> 3;
    const uint32_t per_block = ROWS_THREADS * ROWS_UNROLL;
    dim3 grid((a.total + per_block - 1) / per_block), block(ROWS_THREADS);
    const bool wide = p.sr && spans_counter_words(p.index_base, a.total);
#define MX_ROWS_LAUNCH(T, SR, FL) \
    do { \
        if (wide) hipLaunchKernelGGL((quantize_rows_kernel<T, SR, FL, SR>), grid, block, 0, st, a); \
        else      hipLaunchKernelGGL((quantize_rows_kernel<T, SR, FL, false>), grid, block, 0, st, a); \
    } while (0)
    const int variant = (p.bf16 ? 4 : 0) | (p.sr ? 2 : 0) | (p.floor_mode ? 1 : 0);
    switch (variant) {
        case 0: MX_ROWS_LAUNCH(float, false, false); break;
        case 1: MX_ROWS_LAUNCH(float, false, true); break;
        case 2: MX_ROWS_LAUNCH(float, true, false); break;
        case 3: MX_ROWS_LAUNCH(float, true, true); break;
        case 4: MX_ROWS_LAUNCH(uint16_t, false, false); break;
        case 5: MX_ROWS_LAUNCH(uint16_t, false, true); break;
        case 6: MX_ROWS_LAUNCH(uint16_t, true, false); break;
        default: MX_ROWS_LAUNCH(uint16_t, true, true); break;
    }
#undef MX_ROWS_LAUNCH
    return hipGetLastError();
}

hipError_t launch_quantize_rows_batch(const QuantRowsParams* p, int count, hipStream_t st, const WidenJob* widen)
{
    if (count < 1 || count > 2) return hipErrorInvalidValue;
    RowsBatch b{};
    uint64_t chunks = 0;
    for (int j = 0; j < count; ++j) {
        RowsArgs& a = b.job[j];
        if (p[j].ld != p[j].cols || p[j].sr || p[j].floor_mode != p[0].floor_mode) return hipErrorInvalidValue;
        a.src = p[j].src; a.codes = p[j].codes; a.scales = p[j].scales;
        a.total = (uint32_t)(p[j].rows * (p[j].cols / 8));
        b.bf16[j] = p[j].bf16 ? 1 : 0;
        chunks += a.total;
    }
    // one chunk per lane until that fills the chip's wave slots twice over, then four (loads in flight per lane)
    const bool wide = chunks > 2u * 256u * 2048u;
    const uint32_t per_block = ROWS_THREADS * (wide ? ROWS_UNROLL : 1);
    const uint32_t n0 = (b.job[0].total + per_block - 1) / per_block;
    const uint32_t n1 = count > 1 ? (b.job[1].total + per_block - 1) / per_block : 0u;
    b.first1 = count > 1 ? n0 : 0xFFFFFFFFu;
    uint32_t blocks = n0 + n1;
    if (widen && widen->count) {
        b.widen = *widen;
        ++blocks;
    }
    dim3 grid(blocks), block(ROWS_THREADS);
    if (p[0].floor_mode) {
        if (wide) hipLaunchKernelGGL((quantize_rows_batch_kernel<true, ROWS_UNROLL>), grid, block, 0, st, b);
        else      hipLaunchKernelGGL((quantize_rows_batch_kernel<true, 1>), grid, block, 0, st, b);
    } else {
        if (wide) hipLaunchKernelGGL((quantize_rows_batch_kernel<false, ROWS_UNROLL>), grid, block, 0, st, b);
        else      hipLaunchKernelGGL((quantize_rows_batch_kernel<false, 1>), grid, block, 0, st, b);
    }
    return hipGetLastError();
}

hipError_t launch_quantize_rows_e3m0(const QuantRowsParams& p, hipStream_t st)
{
    RowsArgs a{};
    a.src = p.src; a.codes = p.codes; a.scales = p.scales; a.ema = nullptr;
    a.ld = p.ld; a.cpr = (uint32_t)(p.cols / 8); a.total = (uint32_t)(p.rows * (p.cols / 8));
    a.contiguous = p.ld == p.cols; a.floor_mode = p.floor_mode;
    a.k0 = (uint32_t)p.seed; a.k1 = (uint32_t)(p.seed >> 32); a.tensor_id = p.tensor_id;
    a.base_blk = p.index_base >> 3;
    uint32_t blocks = (a.total + ROWS_THREADS - 1) / ROWS_THREADS;
    dim3 grid(blocks < 8192u ? blocks : 8192u), block(ROWS_THREADS);
#define MX_ROWS_LAUNCH(T, SR, FL) hipLaunchKernelGGL((quantize_rows_e3m0_kernel<T, SR, FL>), grid, block, 0, st, a)
    const int variant = (p.bf16 ? 4 : 0) | (p.sr ? 2 : 0) | (p.floor_mode ? 1 : 0);
    switch (variant) {
        case 0: MX_ROWS_LAUNCH(float, false, false); break;
        case 1: MX_ROWS_LAUNCH(float, false, true); break;
        case 2: MX_ROWS_LAUNCH(float, true, false); break;
        case 3: MX_ROWS_LAUNCH(float, true, true); break;
        case 4: MX_ROWS_LAUNCH(uint16_t, false, false); break;
        case 5: MX_ROWS_LAUNCH(uint16_t, false, true); break;
        case 6: MX_ROWS_LAUNCH(uint16_t, true, false); break;
        default: MX_ROWS_LAUNCH(uint16_t, true, true); break;
    }
#undef MX_ROWS_LAUNCH
    return hipGetLastError();
}

hipError_t launch_dequantize_e3m0(const uint8_t* codes, const uint8_t* scales, int64_t rows, int64_t cols,
                                  float* out, hipStream_t st)
{
    int64_t total = rows * (cols / 2);
    dim3 grid((unsigned)((total + 255) / 256)), block(256);
    hipLaunchKernelGGL(dequantize_e3m0_kernel, grid, block, 0, st, codes, scales, total, cols, out);
    return hipGetLastError();
}

hipError_t launch_ema_quantize(const QuantRowsParams& p, float* ema, float beta, int update_ema, hipStream_t st)
{
    RowsArgs a{};
    a.src = p.src; a.codes = p.codes; a.scales = p.scales; a.ema = ema;
    a.ld = p.ld; a.cpr = (uint32_t)(p.cols / 8); a.total = (uint32_t)(p.rows * (p.cols / 8));
    a.contiguous = p.ld == p.cols; a.floor_mode = p.floor_mode;
    a.beta = beta; a.update_ema = update_ema;
    dim3 grid((a.total + ROWS_THREADS - 1) / ROWS_THREADS), block(ROWS_THREADS);
    if (p.bf16) hipLaunchKernelGGL((ema_quantize_kernel<uint16_t>), grid, block, 0, st, a);
    else        hipLaunchKernelGGL((ema_quantize_kernel<float>), grid, block, 0, st, a);
    return hipGetLastError();
}

template <int SRC, bool FL, bool CS, int WAVES, bool ROW_SR, bool T_SR>
static void launch_tile_wide(const TileBatch& a, bool wide, dim3 grid, hipStream_t st)
{
    dim3 block(64 * WAVES);
    if (wide) hipLaunchKernelGGL((quantize_tile_kernel<SRC, ROW_SR, T_SR, FL, CS, WAVES, ROW_SR || T_SR>), grid, block, 0, st, a);
    else      hipLaunchKernelGGL((quantize_tile_kernel<SRC, ROW_SR, T_SR, FL, CS, WAVES, false>), grid, block, 0, st, a);
}

template <int SRC, bool FL, bool CS, int WAVES>
static void launch_tile_flags(const TileBatch& a, bool row_sr, bool t_sr, bool wide, dim3 grid, hipStream_t st)
{
    if (row_sr) {
        if (t_sr) launch_tile_wide<SRC, FL, CS, WAVES, true, true>(a, wide, grid, st);
        else      launch_tile_wide<SRC, FL, CS, WAVES, true, false>(a, wide, grid, st);
    } else {
        if (t_sr) launch_tile_wide<SRC, FL, CS, WAVES, false, true>(a, wide, grid, st);
        else      launch_tile_wide<SRC, FL, CS, WAVES, false, false>(a, false, grid, st);
    }
}

template <int SRC, bool FL>
static void launch_tile_src(const TileBatch& a, bool row_sr, bool t_sr, bool col_sums, int waves, bool wide, dim3 grid, hipStream_t st)
{
    if constexpr (SRC != 2) {
        if (col_sums) return launch_tile_flags<SRC, FL, true, 8>(a, row_sr, t_sr, wide, grid, st);
    }
    if constexpr (SRC == 0) {
        if (waves == 8) return launch_tile_flags<SRC, FL, false, 8>(a, row_sr, t_sr, wide, grid, st);
    }
    launch_tile_flags<SRC, FL, false, 4>(a, row_sr, t_sr, wide, grid, st);
}

// Waves of a macro tile.  Column sums are kept per 256 rows: eight.  Otherwise four (see above), except for FP32 sources so
// large that memory bounds them: eight waves write the transposed codes in whole lines of 128 bytes.  Four against eight
// waves, in us: deterministic 50432 x 3072 184 / 169, 25216 x 1536 49.2 / 47.2, 12608 x 3072 51.5 / 48.3, below that
// either way (18912 x 2304 53.4 / 54.0, 18912 x 1536 34.9 / 36.7); stochastic column groups, which the vector ALUs bound
// longer, 50432 x 3072 176 / 170, 37824 x 3072 135 / 132, 25216 x 3072 90 / 91, 25216 x 1024 31.9 / 34.3.
static int tile_waves(const QuantTileParams* jobs, int count, bool col_sums)
{
    if (col_sums) return 8;
    int64_t largest = 0;
    for (int j = 0; j < count; ++j) {
        if (jobs[j].row_codes_in || jobs[j].bf16) return 4;
        largest = std::max(largest, jobs[j].rows * jobs[j].cols);
    }
    return largest >= ((int64_t)(jobs[0].sr_t ? 112 : 36) << 20) ? 8 : 4;
}

// How many of a launch's last tiles of 128 columns are issued as their halves of 64: twice the workgroups, half the time.  What
// counts is how evenly the 256 compute units are loaded, also where all tiles run at once: the tiles beyond a multiple of 256
// as halves, up to 128 of them, take 0.87 to 0.97 of the time that they take whole (384 and 768 columns, 264 to 3096 tiles, every
// kind of source and rounding; FP32 with nothing stochastic, which memory bounds, up to 64 only: beyond, 0.95 to 1.07), and up to
// 128 tiles altogether 0.73 to 0.97.  In us, whole / halves / all tiles as halves: bf16 X 282 tiles of 768 columns 9.1 / 7.8 / 8.8,
// 522 12.2 / 10.7 / 12.3, 1068 18.4 / 17.0, 1584 23.5 / 22.0; FP32 X 522 15.1 / 13.7 / 17.2; packed codes 1122 12.7 / 12.0.  With more
// of them it depends on what a round of `slots` tiles that run at once leaves: up to a quarter of a round as halves is even or
// better (FP32 gradient 1470 tiles 33.0 / 31.4; bf16 X 2700 tiles 33.3 / 32.2), except where six waves share a SIMD and all tiles run
// at once whole and not as halves (1409 to 1536 tiles; 1503 of bf16 with both outputs deterministic 16.1 / 18.8).
static uint32_t tile_tail(uint32_t n_tiles, uint32_t slots, uint32_t at_once, bool plain_f32)
{
    const uint32_t over = n_tiles % 256u, rem = n_tiles % slots;
    if (over <= (plain_f32 && n_tiles > 256u ? 64u : 128u)) return over;
    if (rem > slots / 4u || (n_tiles <= at_once && n_tiles + rem > at_once)) return 0u;
    return rem;
}

// Fills the kernel arguments of one tensor; returns its number of workgroups.
static uint32_t make_tile_args(const QuantTileParams& p, int waves, int per_simd, TileArgs& a)
{
    a = TileArgs{};
    a.src = p.src; a.row_codes_in = p.row_codes_in; a.row_scales_in = p.row_scales_in;
    a.codes_t = p.codes_t; a.scales_t = p.scales_t; a.codes_row = p.codes_row; a.scales_row = p.scales_row;
    a.ld = p.ld; a.rows = (uint32_t)p.rows; a.cols = (uint32_t)p.cols;
    a.src_rows = p.src_rows ? (uint32_t)p.src_rows : (uint32_t)p.rows; a.src_bf16 = p.bf16 ? 1 : 0;
    a.pre_quant = p.pre_quant; a.want_row = p.codes_row != nullptr;
    a.k0 = (uint32_t)p.seed; a.k1 = (uint32_t)(p.seed >> 32);
    a.seed_dev = reinterpret_cast<const uint32_t*>(p.seed_dev);
    a.col_sum_partials = p.col_sums ? p.col_sum_workspace : nullptr;
    a.tensor_id_t = p.tensor_id_t; a.tensor_id_row = p.tensor_id_row; a.index_base = p.index_base;
    const uint32_t wide_per_row = (uint32_t)((p.cols + 127) / 128);
    const uint32_t macro_rows = 32u * (uint32_t)waves, at_once = 256u * 4u * (uint32_t)per_simd / (uint32_t)waves;
    const uint32_t slots = per_simd == 6 ? at_once / 6u * 5u : at_once;         // a sixth wave gains nothing at the quarter of a round
    const uint32_t n_tiles = (uint32_t)((p.rows + macro_rows - 1) / macro_rows) * wide_per_row;
    const uint32_t n_wide = n_tiles - tile_tail(n_tiles, slots, at_once, !p.bf16 && !p.row_codes_in && !p.sr_t && !p.sr_row);
    a.n_wide = n_wide; a.wide_per_row = wide_per_row;
    return n_wide + 2u * (n_tiles - n_wide);
}

uint32_t tile_workgroups(int64_t rows, int64_t cols, int src, bool row_sr, bool t_sr)
{
    QuantTileParams p{};
    TileArgs a;
    p.rows = rows; p.cols = cols; p.bf16 = src == 1; p.sr_row = row_sr; p.sr_t = t_sr;
    return make_tile_args(p, 4, tile_waves_per_simd(src, row_sr, t_sr, 4), a);
}

hipError_t launch_quantize_tile_batch(const QuantTileParams* jobs, int count, hipStream_t st, const WidenJob* widen,
                                      bool finish_col_sums)
{
    if (count < 1 || count > TILE_BATCH_MAX) return hipErrorInvalidValue;
    const QuantTileParams& p = jobs[0];
    const bool row_sr = p.row_codes_in ? false : p.sr_row;
    TileBatch b{};
    uint32_t blocks = 0;
    bool col_sums = false, mixed = false, wide = false;
    for (int j = 0; j < count; ++j) {
        col_sums = col_sums || jobs[j].col_sums != nullptr;
        mixed = mixed || (!p.row_codes_in && jobs[j].bf16 != p.bf16);
    }
    const int waves = tile_waves(jobs, count, !p.row_codes_in && col_sums);
    const int per_simd = tile_waves_per_simd(p.row_codes_in ? 2 : p.bf16 && !mixed ? 1 : 0, row_sr, p.sr_t, waves);
    for (int j = 0; j < TILE_BATCH_MAX; ++j) {
        b.first[j] = 0xFFFFFFFFu;
        if (j >= count) continue;
        const QuantTileParams& q = jobs[j];
        // one kernel instance serves the launch: kind of source, roundings and scale rule are shared
        if ((q.row_codes_in != nullptr) != (p.row_codes_in != nullptr) || q.sr_t != p.sr_t ||
            (q.row_codes_in ? false : q.sr_row) != row_sr || q.floor_mode != p.floor_mode)
            return hipErrorInvalidValue;
        b.first[j] = blocks;
        blocks += make_tile_args(q, waves, per_simd, b.job[j]);
        wide = wide || spans_counter_words(q.index_base, (uint64_t)q.rows * (uint64_t)(q.cols / 8));
    }
    if (mixed && (col_sums || row_sr)) return hipErrorInvalidValue;      // only the forward pass mixes source types
    if (widen && widen->count) {
        b.widen = *widen;
        ++blocks;
    }
    dim3 grid(blocks);
    const int src = p.row_codes_in ? 2 : mixed ? 3 : p.bf16 ? 1 : 0;
    auto launch = [&](auto fl) {
        constexpr bool FL = decltype(fl)::value;
        switch (src) {
            case 0: launch_tile_src<0, FL>(b, row_sr, p.sr_t, col_sums, waves, wide, grid, st); break;
            case 1: launch_tile_src<1, FL>(b, row_sr, p.sr_t, col_sums, waves, wide, grid, st); break;
            case 2: launch_tile_src<2, FL>(b, row_sr, p.sr_t, false, waves, wide, grid, st); break;
            default:
                if (p.sr_t) launch_tile_wide<3, FL, false, 4, false, true>(b, wide, grid, st);
                else        launch_tile_wide<3, FL, false, 4, false, false>(b, false, grid, st);
        }
    };
    if (p.floor_mode) launch(std::true_type{});
    else              launch(std::false_type{});
    hipError_t e = hipGetLastError();
    for (int j = 0; j < count && e == hipSuccess && finish_col_sums; ++j)
        if (jobs[j].col_sums) e = launch_column_sum_finish(column_sum_tail(jobs[j]), st);
    return e;
}

ColumnSumTail column_sum_tail(const QuantTileParams& q)
{
    return {q.col_sum_workspace, q.col_sums, (uint32_t)((q.rows + 255) / 256), (uint32_t)q.cols, q.col_sums_bf16 ? 1 : 0};
}

hipError_t launch_column_sum_finish(const ColumnSumTail& t, hipStream_t st)
{
    hipLaunchKernelGGL(column_sum_finish_kernel, dim3((t.cols + 31) / 32), dim3(256), 0, st, t);
    return hipGetLastError();
}

size_t column_sum_workspace_bytes(int64_t rows, int64_t cols)
{
    return (size_t)((rows + 255) / 256) * (size_t)cols * sizeof(float);
}

hipError_t launch_quantize_tile(const QuantTileParams& p, hipStream_t st)
{
    return launch_quantize_tile_batch(&p, 1, st, nullptr, true);
}

hipError_t launch_calibration_copy(void* dst, const void* src, size_t bytes, hipStream_t st)
{
    size_t n = bytes / 16;
    size_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(calibration_copy_kernel, dim3((unsigned)blocks), dim3(256), 0, st,
                       static_cast<const uint4*>(src), static_cast<uint4*>(dst), n);
    return hipGetLastError();
}

hipError_t launch_oscillation(const OscillationParams& p, hipStream_t st)
{
    OscArgs a{};
    a.w = p.w; a.codes = p.codes; a.scales = p.scales; a.w_prev = p.w_prev;
    a.codes_prev = p.codes_prev; a.scales_prev = p.scales_prev; a.dist_w = p.dist_w; a.dist_q = p.dist_q;
    a.ld = p.ld; a.cpr = (uint32_t)(p.cols / 8); a.total = (uint32_t)(p.rows * (p.cols / 8)); a.init = p.init;
    dim3 grid((a.total + ROWS_THREADS - 1) / ROWS_THREADS), block(ROWS_THREADS);
    if (p.bf16) hipLaunchKernelGGL(oscillation_kernel<uint16_t>, grid, block, 0, st, a);
    else        hipLaunchKernelGGL(oscillation_kernel<float>, grid, block, 0, st, a);
    return hipGetLastError();
}

hipError_t launch_confidence(const ConfidenceParams& p, hipStream_t st)
{
    ConfArgs a{};
    a.w = p.w; a.conf = p.conf; a.hist = reinterpret_cast<unsigned long long*>(p.hist); a.ld = p.ld;
    a.cpr = (uint32_t)(p.cols / 8); a.total = (uint32_t)(p.rows * (p.cols / 8));
    a.bins = p.hist ? p.bins : 0; a.floor_mode = p.floor_mode;
    // at most one workgroup per compute unit: each one flushes its histogram to memory once
    uint32_t blocks = (a.total + ROWS_THREADS - 1) / ROWS_THREADS;
    dim3 grid(blocks < 256u ? blocks : 256u), block(ROWS_THREADS);
    if (p.bf16) hipLaunchKernelGGL(confidence_kernel<uint16_t>, grid, block, 0, st, a);
    else        hipLaunchKernelGGL(confidence_kernel<float>, grid, block, 0, st, a);
    return hipGetLastError();
}

size_t rate_workspace_bytes() { return (size_t)RATE_BLOCKS * 2 * sizeof(double); }

hipError_t launch_rate_of_change(const RateParams& p, hipStream_t st)
{
    RateArgs a{};
    a.x = p.x; a.x_prev = p.x_prev; a.partial = p.partial; a.ld = p.ld;
    a.cpr = (uint32_t)(p.cols / 8); a.total = (uint32_t)(p.rows * (p.cols / 8)); a.init = p.init;
    dim3 grid(RATE_BLOCKS), block(ROWS_THREADS);
    if (p.bf16) hipLaunchKernelGGL(rate_partial_kernel<uint16_t>, grid, block, 0, st, a);
    else        hipLaunchKernelGGL(rate_partial_kernel<float>, grid, block, 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(rate_finish_kernel, dim3(1), block, 0, st, p.partial, p.init, p.result);
    return hipGetLastError();
}

hipError_t launch_ramping_factor(const float* dist_w, const float* dist_q, int64_t count, float k1, int k2,
                                 int n_max, int32_t* factor, hipStream_t st)
{
    dim3 grid((unsigned)((count + 255) / 256)), block(256);
    hipLaunchKernelGGL(ramping_factor_kernel, grid, block, 0, st, dist_w, dist_q, count, k1, k2, n_max, factor);
    return hipGetLastError();
}

hipError_t launch_dequantize(const uint8_t* codes, const uint8_t* scales, int64_t rows, int64_t cols,
                             float* out, hipStream_t st)
{
    int64_t total = rows * (cols / 2);
    dim3 grid((unsigned)((total + 255) / 256)), block(256);
    hipLaunchKernelGGL(dequantize_kernel, grid, block, 0, st, codes, scales, total, cols, out);
    return hipGetLastError();
}

}  // namespace mxl
