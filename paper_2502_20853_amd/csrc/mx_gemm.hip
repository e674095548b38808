// C[m x n] = A[m x k] . B[n x k]^T on packed MXFP4 operands, FP32 accumulation on gfx950's
// block-scaled FP4 matrix cores.  All three products of the layer (Eqs. 3-5, Sec. 3.3) have
// this form because every operand is stored along its own contraction dimension.
//
// Two kernels, chosen by plan_gemm (plan_fused for products with the GELU stage) at the end of the file:
//   mx_gemm_pingpong_kernel  the main path (K a multiple of 128, at least 4 K steps per K split;
//       every ViT-B/L product): one persistent workgroup of 8 waves per compute unit, tile 256 x 256,
//       operands global -> LDS by DMA loads, two wave groups alternating between their MFMA burst and
//       their LDS/DMA work.  Described in full above the kernel.
//   mx_gemm_tile_kernel      any K that is a multiple of 32, any size: one tile (128 x 128, 128 x 64 or 64 x 64)
//       per workgroup of 4 waves, register-staged loads, zero-filled K tail.  Smaller products, short or ragged K.
// A K-split product (dW: K = tokens, small output) writes FP32 partials to the caller's workspace
// and splitk_reduce*_kernel adds them in a fixed order.
//
// Common to both:
//   - V_MFMA_SCALE_F32_32X32X64_F8F6F4: it consumes, per lane, 32 consecutive K elements (16 bytes, exactly one
//     MX group) of one row and that group's E8M0 scale byte (row lane % 32, K block lane / 32);
//   - code tiles sit in LDS row-major with the 16-byte chunk index XOR-swizzled by the row (by (row >> 2) & 3
//     at 64 bytes per row), so that both the 16-byte writes and the MFMA operand reads (one chunk of 32 rows)
//     are bank-conflict free;
//   - the MFMA's first operand is the B (n) side, so that a lane ends up with runs of four
//     consecutive n of one m and stores 8 or 16 contiguous bytes.
#include "mx_device.hpp"
#include "mx_launch.hpp"

#include <algorithm>
#include <cmath>
#include <type_traits>

// Timing hooks for instrumented builds of this file (a build that defines them before including it);
// they expand to nothing in the library.
#ifndef MX_PROBE
#define MX_PROBE_INIT
#define MX_PROBE(id)
#endif

namespace {

// compile-time loop: the MFMA's op_sel (which scale byte) must be an immediate
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

struct GemmArgs {
    const uint8_t* a_codes;
    const uint8_t* a_scales;
    const uint8_t* b_codes;
    const uint8_t* b_scales;
    uint32_t m, n, k;        // k in elements
    uint32_t k_per_split;    // multiple of 128
    void* c;                 // final output, or FP32 partials [split][m][n] when split_k > 1
    int64_t ldc;
    int c_bf16;
    int split_k;
    uint32_t tiles_m, tiles_n;
    int stagger;             // start delay of every other workgroup of an XCD, in s_sleep(32) units
    const float* bias;       // n values added to every row of a final output (n % 4 == 0), or null
    uint8_t* q_codes;        // fused GELU + 1x32 quantizer of the output rows: packed codes
    uint8_t* q_scales;       //   [m x n/2] and scale bytes [m x n/32] of Q(GELU(product + bias)), or null
    int q_floor;             //   its scale rule: 0 truncation-free, 1 Eq. 2
};

// FP32 -> bf16, round to nearest even, with gfx950's packed convert instruction.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t f32x2_to_bf16x2(float lo, float hi)
{
    f32x2_t v = {lo, hi};
    bf16x2_t b = __builtin_convertvector(v, bf16x2_t);
    return *reinterpret_cast<uint32_t*>(&b);
}

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f)
{
    return (uint16_t)f32x2_to_bf16x2(f, 0.f);
}

typedef float v16f __attribute__((ext_vector_type(16)));

// 16-byte store.  A final output is written with the nontemporal hint (by the tile kernels where stream_output says so): it
// is not read again here, and without the hint an output larger than the last-level cache slows the whole kernel
// down while it drains (split-K partials keep the default policy, the reduction reads them).
template <bool STREAM>
__device__ __forceinline__ void store16(void* dst, v4i v)
{
    if (STREAM) __builtin_nontemporal_store(v, reinterpret_cast<v4i*>(dst));
    else        *reinterpret_cast<v4i*>(dst) = v;
}

// Workgroup -> (K split, tile).  The grid is one-dimensional over split * tiles.  Workgroup
// ids go round-robin over the 8 XCDs, each with its own L2, so id % 8 = XCD gets a
// contiguous range of the logical order (split, m tile, n tile): the workgroups that share
// an A row panel or a B panel of one K range run on the same XCD at about the same time.
__device__ __forceinline__ void decode_tile(const GemmArgs& g, uint32_t bid, uint32_t& zsplit, uint32_t& tm, uint32_t& tn)
{
    const uint32_t tiles = g.tiles_m * g.tiles_n, nblk = tiles * (uint32_t)g.split_k;
    uint32_t per = nblk / 8, rem = nblk % 8;
    uint32_t xcd = bid % 8, idx = bid / 8;
    bid = xcd * per + (xcd < rem ? xcd : rem) + idx;       // bijection on [0, nblk)
    zsplit = bid / tiles;
    uint32_t t = bid - zsplit * tiles;
    tm = t / g.tiles_n;
    tn = t - tm * g.tiles_n;
}

// Four consecutive scale bytes [off, off + 4) of a row that starts `left` bytes before the end of the
// scale array; the address has no alignment.  Bytes past the end of the array are not read (they belong
// to K groups whose codes are zero; any other byte there is some row's scale, never the NaN code 255).
__device__ __forceinline__ uint32_t load_scales4(const uint8_t* row, uint32_t off, uint32_t left)
{
    uint32_t v = 0u;
    if (off + 4u <= left) {
        __builtin_memcpy(&v, row + off, 4);
    } else {
        for (uint32_t b = 0; b < 4; ++b)
            if (off + b < left) v |= (uint32_t)row[off + b] << (8 * b);
    }
    return v;
}

// ---------------------------------------------------------------------------
// Products that the main kernel does not take: any K that is a multiple of 32, any m and n.
//
//   workgroup 4 waves (2 x 2), tile BM x BN, wave tile BM/2 x BN/2 of 32 x 32 x 64 MFMA tiles; K step KS.
//   Operands go global -> registers -> LDS, the next step's loads in flight during the current step's
//   MFMAs; chunks past the end of K are zero-filled in registers, so K needs no alignment beyond a group.
//   (No DMA loads: they cannot zero-fill a ragged K tail, and scale rows of K/32 bytes have no alignment.)
// Shapes (chosen in plan_gemm, which gives the times):
//   128 x 128, KS 128 (384, one step, for K up to that): 35 KB (52) of LDS, three workgroups per compute unit, so that one
//     stores its tile or waits for its first loads while the others multiply; at four, the 128 registers allowed spill,
//     which took half as long again.
//   128 x 64, KS 256: half the tile and twice the K step, for products with fewer tiles, where the latency of a
//     K step counts (12608 x 192 x 768: 6.3 us against 7.4).
//   64 x 64, KS 512: for products too small to fill the chip otherwise.  What such a launch costs is the chain
//     launch -> first load -> multiply -> store; a K step of 512 puts all operand loads of a K <= 512 product in
//     flight at once instead of one latency per 128.  A second K step in flight (two register sets) gained
//     nothing: the step is a chain of LDS writes, barrier, LDS reads and eight dependent MFMAs, 0.9 us.
// ---------------------------------------------------------------------------
constexpr int T_NT = 256;

template <int BM_, int BN_, int KS_, int OCC_>
struct TileShape {
    static constexpr int BM = BM_, BN = BN_, KS = KS_, OCC = OCC_;   // OCC: workgroups per compute unit
    static constexpr int ROWB = KS / 2;                         // code bytes of a row and K step
    static constexpr int PITCH = ROWB;
    static constexpr int SCALEB = KS / 32;
    static constexpr int SPITCH = SCALEB + (KS % 256 == 0 ? 4 : 0);   // KS 128 and 384: 1 and 3 dwords per row, conflict-free as they are
    static constexpr int STAGE = (BM + BN) * (PITCH + SPITCH);
    static constexpr int STAGES = KS == 384 ? 1 : 2;            // one: K <= KS, a single step
    static constexpr int EP_PITCH = BN / 2 * 4 + 16;            // output strip: 32 rows of BN/2 FP32 values
    static constexpr int LDS = STAGES * STAGE > 4 * 32 * EP_PITCH ? STAGES * STAGE : 4 * 32 * EP_PITCH;
    // 16-byte column of a chunk: XOR-swizzled, so that the 16 lanes of an access phase (16 rows of one chunk, or
    // 4 to 16 chunks of a row) spread over all banks
    static __device__ __forceinline__ uint32_t column(uint32_t row, uint32_t chunk)
    {
        if (KS == 384) {                                        // 12 chunks: rotated instead
            const uint32_t p = chunk + ((row >> 2) & 3u);
            return (p >= 12u ? p - 12u : p) << 4;
        }
        return (KS == 128 ? chunk ^ ((row >> 2) & 3u) : KS == 256 ? chunk ^ ((row >> 1) & 7u) : chunk ^ (row & 15u)) << 4;
    }
};

typedef __attribute__((address_space(3))) uint8_t lds_u8;

// Lanes of a wave hand values to each other through its LDS strip: what is written before this call is seen by every lane's
// reads after it, and what is read before it was not yet overwritten.  It takes no instruction, because the LDS executes a
// wave's instructions in order; it keeps the compiler from moving the accesses past each other.
__device__ __forceinline__ void strip_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
}

// The output stage of a wave whose TI x TJ tiles of 32 x 32 lie wholly inside the matrix, with rows that can be stored 16
// bytes at a time: no bounds tests, a store's address is a uniform pointer plus one lane offset, and the strip's
// accesses need no waits (the LDS executes a wave's instructions in order), so 32 rows are converted and written to the
// strip while the stores of the 32 before them are issued.  A short-K product is bound by this stage (25216 x 1536 FP32:
// 155 MB): against the form with tests below, 25216 x 1152 x 384 bf16 21.5 -> 19.4 us, 50432 x 768 x 192 22.2 -> 19.6.
template <int TI, int TJ, bool STREAM, bool BF16>
__device__ __forceinline__ void tile_epilogue_interior(const GemmArgs& g, lds_u8* ep, v16f (&acc)[TI][TJ], uint32_t mrow0,
                                                       uint32_t nbase, uint32_t zsplit, int64_t ldc)
{
    typedef __attribute__((address_space(3))) v4i lds_v4i;
    typedef __attribute__((address_space(3))) v4f lds_v4f;
    typedef int v2i __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(3))) v2i lds_v2i;
    constexpr int ES = BF16 ? 2 : 4, COLS = 32 * TJ, PITCH = COLS * 4 + 16, LPR = COLS * ES / 16, RPI = 64 / LPR, STORES = 32 / RPI;
    const uint32_t lane = threadIdx.x & 63, lrow = lane & 31, lhalf = lane >> 5;
    uint8_t* base = static_cast<uint8_t*>(g.c);
    if (!BF16 && g.split_k > 1) base += (size_t)zsplit * g.m * g.n * 4;
    uint8_t* tile = base + ((size_t)mrow0 * ldc + nbase) * ES;                            // uniform
    const uint32_t voff = (lane / LPR) * (uint32_t)ldc * ES + (lane % LPR) * 16;
    lds_u8* wr = ep + lrow * PITCH + lhalf * 4 * ES;
    const lds_u8* rd = ep + (lane / LPR) * PITCH + (lane % LPR) * 16;
    v4f bias[TJ][4];
    if (g.bias != nullptr) {
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) bias[j][q] = *reinterpret_cast<const v4f*>(g.bias + nbase + 32 * j + 8 * q + 4 * lhalf);
    }
    auto write_rows = [&](int i) {
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v4f v = v4f{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                if (g.bias != nullptr) v += bias[j][q];
                if (BF16) *reinterpret_cast<lds_v2i*>(wr + (32 * j + 8 * q) * 2) = v2i{(int)f32x2_to_bf16x2(v.x, v.y), (int)f32x2_to_bf16x2(v.z, v.w)};
                else      *reinterpret_cast<lds_v4f*>(wr + (32 * j + 8 * q) * 4) = v;
            }
    };
    write_rows(0);
#pragma unroll
    for (int i = 0; i < TI; ++i) {
        v4i v[STORES];
        strip_order();
#pragma unroll
        for (int it = 0; it < STORES; ++it) v[it] = *reinterpret_cast<const lds_v4i*>(rd + it * RPI * PITCH);
        strip_order();
        if (i + 1 < TI) write_rows(i + 1);
#pragma unroll
        for (int it = 0; it < STORES; ++it) store16<STREAM>(tile + (size_t)(i * 32 + it * RPI) * ldc * ES + voff, v[it]);
    }
}

// Accumulators of one wave (TI x TJ tiles of 32 x 32; first row mrow0, first column nbase) through a per-wave
// LDS strip of 32 rows, so that a store instruction writes 16 bytes per lane and whole row segments.
template <int TI, int TJ, bool STREAM>
__device__ __forceinline__ void tile_epilogue(const GemmArgs& g, uint8_t* ep, v16f (&acc)[TI][TJ], uint32_t mrow0,
                                              uint32_t nbase, uint32_t zsplit)
{
    constexpr int COLS = 32 * TJ, PITCH = COLS * 4 + 16;
    const uint32_t lane = threadIdx.x & 63, lrow = lane & 31, lhalf = lane >> 5;
    float* cf = static_cast<float*>(g.c);
    uint16_t* ch = static_cast<uint16_t*>(g.c);
    int64_t ldc = g.ldc;
    if (g.split_k > 1) {
        cf += (size_t)zsplit * g.m * g.n;
        ldc = g.n;
    }
    const bool as_bf16 = g.c_bf16 && g.split_k == 1;
    const bool vec_ok = as_bf16 ? (ldc & 7) == 0 && (reinterpret_cast<uintptr_t>(ch) & 15) == 0
                                : (ldc & 3) == 0 && (reinterpret_cast<uintptr_t>(cf) & 15) == 0;
    if (mrow0 + 32 * TI <= g.m && nbase + 32 * TJ <= g.n && vec_ok && ldc < (1 << 26)) {       // uniform
        if (as_bf16) tile_epilogue_interior<TI, TJ, STREAM, true>(g, (lds_u8*)ep, acc, mrow0, nbase, zsplit, ldc);
        else         tile_epilogue_interior<TI, TJ, STREAM, false>(g, (lds_u8*)ep, acc, mrow0, nbase, zsplit, ldc);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        return;
    }
#pragma unroll
    for (int i = 0; i < TI; ++i) {
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t col = 32 * j + 8 * q + 4 * lhalf;
                v4f v = v4f{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                if (g.bias != nullptr && nbase + col < g.n) v += *reinterpret_cast<const v4f*>(g.bias + nbase + col);   // n % 4 == 0
                if (as_bf16) {
                    uint2 pk;
                    pk.x = f32x2_to_bf16x2(v.x, v.y);
                    pk.y = f32x2_to_bf16x2(v.z, v.w);
                    *reinterpret_cast<uint2*>(ep + lrow * PITCH + col * 2) = pk;
                } else {
                    *reinterpret_cast<v4f*>(ep + lrow * PITCH + col * 4) = v;
                }
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (as_bf16) {
            constexpr int LPR = COLS / 8, RPI = 64 / LPR;          // lanes per row, rows per instruction
#pragma unroll
            for (int it = 0; it < 32 / RPI; ++it) {
                const uint32_t row = it * RPI + lane / LPR, col = (lane % LPR) * 8;
                const uint32_t mm = mrow0 + i * 32 + row, nn = nbase + col;
                const v4i v = *reinterpret_cast<const v4i*>(ep + row * PITCH + col * 2);
                if (mm < g.m && nn < g.n) {
                    uint16_t* dst = ch + (size_t)mm * ldc + nn;
                    if (nn + 8 <= g.n && vec_ok) {
                        store16<STREAM>(dst, v);
                    } else {
                        for (int e = 0; e < 8; ++e)
                            if (nn + e < g.n) dst[e] = (uint16_t)((uint32_t)v[e >> 1] >> (16 * (e & 1)));
                    }
                }
            }
        } else {
            constexpr int LPR = COLS / 4, RPI = 64 / LPR;
#pragma unroll
            for (int it = 0; it < 32 / RPI; ++it) {
                const uint32_t row = it * RPI + lane / LPR, col = (lane % LPR) * 4;
                const uint32_t mm = mrow0 + i * 32 + row, nn = nbase + col;
                const v4i v = *reinterpret_cast<const v4i*>(ep + row * PITCH + col * 4);
                if (mm < g.m && nn < g.n) {
                    float* dst = cf + (size_t)mm * ldc + nn;
                    if (nn + 4 <= g.n && vec_ok) {
                        store16<STREAM>(dst, v);
                    } else {
                        for (int e = 0; e < 4; ++e)
                            if (nn + e < g.n) dst[e] = __int_as_float(v[e]);
                    }
                }
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
}

// GELU(x) = x * Phi(x) with Phi(x) = erfc(-x / sqrt(2)) / 2 (the exact form, not the tanh approximation),
// FP32, branch-free, 26 instructions.  With z = |x| / sqrt(2):
//     erfc(z) = exp(-z^2) * G(z),   G(z) = t * P8(t - t0),   t = 1 / (1 + z / 2),
// where P8 is a degree-8 fit of the scaled complementary error function over z in [0, 12.1] (relative error
// 4.4e-8 in exact arithmetic; coefficients from fit_gelu_erfcx.py beside the package's Python files).
// erfc keeps its relative accuracy in the negative tail, where 1 + erf would cancel; to keep it through the
// exponential, z^2 = x^2 / 2 is carried as an FP32 product and its exact remainder, and the exponent of two as
// a rounded product and its remainder, both folded in as first-order corrections.  Against the FP64 value the
// result is within 4.8e-7 |GELU(x)| (2^-18 is 3.8e-6) for every x where |GELU(x)| >= 2^-100, and below
// 2^-120 in absolute terms beyond (checked on 6e6 points by the fitting script's FP32 emulation).  |x| is
// clamped at 17 before squaring: erfc has long underflowed there, and no infinity can arise.
//
// The operation sequence of float gelu_f32(float x) as the fitting script emulates it, four values side by side: the stage
// is bound by the vector ALUs, two waves share a SIMD, and one dependent chain per value (two of its instructions
// transcendental) leaves it idle.  25216 x 3072 x 768 on the main kernel: 150 us value by value with 30 instructions each
// and codes packed by shifts, 140 in this form; on 128 x 128 tiles 110 to 125 (the product alone takes 45).
__device__ __forceinline__ void gelu4_f32(const float (&x)[4], float (&y)[4])
{
    constexpr float T0 = 0.5709219574928284f;
    constexpr float C0 = 0.562385082244873f, C1 = 0.768385112285614f, C2 = 0.584431529045105f,
                    C3 = 0.09252145141363144f, C4 = -0.20070798695087433f, C5 = -0.058531392365694046f,
                    C6 = 0.11107011884450912f, C7 = 0.014878340996801853f, C8 = -0.05936833471059799f;
    constexpr float C[9] = {C0, C1, C2, C3, C4, C5, C6, C7, C8};
    constexpr float HALF_LOG2E_HI = 0.72134751f;                    // log2(e) / 2 rounded to FP32 ...
    constexpr float HALF_LOG2E_LO = (float)(0.72134752044448170368 - (double)HALF_LOG2E_HI);   // ... and what it lost
    float ax[4], t[4], w[4], g[4], s[4], e[4], c[4], yl[4];
    auto each = [](auto&& f) {
#pragma unroll
        for (int i = 0; i < 4; ++i) f(i);
        __builtin_amdgcn_sched_barrier(0);                          // the four stay side by side
    };
    each([&](int i) { ax[i] = __builtin_fminf(__builtin_fabsf(x[i]), 17.0f); });
    each([&](int i) { t[i] = __builtin_fmaf(ax[i], 0.35355339059327376f, 1.0f); });
    each([&](int i) { t[i] = __builtin_amdgcn_rcpf(t[i]); });                                       // 1 / (1 + z / 2)
    each([&](int i) { s[i] = __fmul_rn(ax[i], ax[i]); });
    each([&](int i) { e[i] = __fmul_rn(s[i], -HALF_LOG2E_HI); });                                   // -yh
    each([&](int i) { yl[i] = __builtin_fmaf(s[i], HALF_LOG2E_HI, e[i]); });        // z^2 log2(e) = yh + yl + r log2(e) / 2 (to first order)
    each([&](int i) { yl[i] = __builtin_fmaf(s[i], HALF_LOG2E_LO, yl[i]); });
    each([&](int i) { e[i] = __builtin_amdgcn_exp2f(e[i]); });
    each([&](int i) { c[i] = __builtin_fmaf(yl[i], -0.34657359f, 0.5f); });                         // 2^-yl / 2
    each([&](int i) { s[i] = __builtin_fmaf(ax[i], ax[i], -s[i]); });                               // r: x^2 = s + r exactly
    each([&](int i) { c[i] = __builtin_fmaf(s[i], -0.25f, c[i]); });                                // exp(-r / 2) / 2
    each([&](int i) { w[i] = t[i] - T0; });
    each([&](int i) { g[i] = __builtin_fmaf(C[8], w[i], C[7]); });
#pragma unroll
    for (int k = 6; k >= 0; --k) each([&](int i) { g[i] = __builtin_fmaf(g[i], w[i], C[k]); });
    each([&](int i) { g[i] = __fmul_rn(g[i], t[i]); });
    each([&](int i) { g[i] = __fmul_rn(g[i], e[i]); });
    each([&](int i) { g[i] = __fmul_rn(g[i], c[i]); });                                             // erfc / 2
    // x Phi(|x|) = x - x erfc / 2 for x >= 0, -|x| erfc / 2 below; the maximum with -0 keeps a zero result's sign
    each([&](int i) { asm("v_max_f32_e32 %0, %1, %2" : "=v"(y[i]) : "v"(x[i]), "v"(-0.0f)); });
    each([&](int i) { y[i] = __builtin_fmaf(-__builtin_fabsf(x[i]), g[i], y[i]); });
}

// The tile kernel's second output stage: the next layer's forward quantizer applied to GELU(product + bias) from the FP32
// accumulators (see gemm_epilogue_gelu_quant for the layout of a lane's values).  Codes go through the wave's strip
// ([32 * TI rows], 16 * TJ bytes each) and leave as 16-byte pieces, then the scale bytes, TJ per row.
template <bool FLOOR, int TI, int TJ>
__device__ __forceinline__ void tile_gelu_quant(const GemmArgs& g, uint8_t* ep, v16f (&acc)[TI][TJ], uint32_t mrow0, uint32_t nbase)
{
    constexpr int PITCH = 16 * TJ + 16, SCALES = 32 * TI * PITCH;
    const uint32_t lane = threadIdx.x & 63, lrow = lane & 31, lhalf = lane >> 5;
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
        v4f bias[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)                                                     // n % 32 == 0
            bias[q] = nbase + 32 * j < g.n ? *reinterpret_cast<const v4f*>(g.bias + nbase + 32 * j + 8 * q + 4 * lhalf) : v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < TI; ++i) {
            float v[16];
            uint32_t m = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float pre[4], post[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) pre[r] = acc[i][j][4 * q + r] + bias[q][r];
                gelu4_f32(pre, post);
#pragma unroll
                for (int r = 0; r < 4; ++r) v[4 * q + r] = post[r];
                m = mxd::absmax3_bits(v[4 * q], v[4 * q + 1], m);
                m = mxd::absmax3_bits(v[4 * q + 2], v[4 * q + 3], m);
            }
            const auto sw = __builtin_amdgcn_permlane32_swap(m, m, false, false);
            m = sw[0] > sw[1] ? sw[0] : sw[1];
            const uint32_t byte = mxd::scale_byte(m, FLOOR);
            const float scale = mxd::scale_operand(byte);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t pk = mxd::cvt_rtn_f32<0>(0u, v[4 * q], v[4 * q + 1], scale);
                pk = mxd::cvt_rtn_f32<1>(pk, v[4 * q + 2], v[4 * q + 3], scale);
                *reinterpret_cast<uint16_t*>(ep + (i * 32 + lrow) * PITCH + 16 * j + 4 * q + 2 * lhalf) = (uint16_t)pk;
            }
            if (lhalf == 0) ep[SCALES + (i * 32 + lrow) * TJ + j] = (uint8_t)byte;
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // the strip is read through other lanes' addresses
    const uint32_t half_n = g.n >> 1, grp_n = g.n >> 5;
    constexpr int RPI = 64 / TJ;                                // rows per instruction
    const uint32_t piece = lane % TJ;
#pragma unroll
    for (int it = 0; it < (32 * TI + RPI - 1) / RPI; ++it) {
        const uint32_t row = it * RPI + lane / TJ;
        if (row < 32 * TI && mrow0 + row < g.m && nbase + 32 * piece < g.n) {
            const v4i c = *reinterpret_cast<const v4i*>(ep + row * PITCH + piece * 16);
            *reinterpret_cast<v4i*>(g.q_codes + (size_t)(mrow0 + row) * half_n + (nbase >> 1) + piece * 16) = c;
        }
    }
    if (lane < 32 * TI && mrow0 + lane < g.m) {
#pragma unroll
        for (int j = 0; j < TJ; ++j)
            if (nbase + 32 * j < g.n) g.q_scales[(size_t)(mrow0 + lane) * grp_n + (nbase >> 5) + j] = ep[SCALES + lane * TJ + j];
    }
}

// One K step of a wave: its TI x TJ tiles from the staged operands at st; `left` K elements are not multiplied yet.
template <typename S, int TI, int TJ>
__device__ __forceinline__ void tile_multiply(const uint8_t* st, uint32_t left, v16f (&acc)[TI][TJ], int wm, int wn, uint32_t lrow, uint32_t lhalf)
{
    constexpr int BM = S::BM, BN = S::BN;
    const uint8_t* pa = st + (wm * (BM / 2) + lrow) * S::PITCH;
    const uint8_t* pb = st + (BM + wn * (BN / 2) + lrow) * S::PITCH;
    const uint8_t* sa = st + (BM + BN) * S::PITCH + (wm * (BM / 2) + lrow) * S::SPITCH;
    const uint8_t* sb = st + (BM + BN) * S::PITCH + (BM + wn * (BN / 2) + lrow) * S::SPITCH;
    static_for<0, S::KS / 128>([&](auto dc) {
        constexpr int d = decltype(dc)::value;
        if (d * 128u >= left) return;                              // uniform: whole 128-K blocks past the end are skipped
        uint32_t ua[TI], ub[TJ];
#pragma unroll
        for (int i = 0; i < TI; ++i) ua[i] = *reinterpret_cast<const uint32_t*>(sa + i * 32 * S::SPITCH + d * 4) >> 8 * lhalf;
#pragma unroll
        for (int j = 0; j < TJ; ++j) ub[j] = *reinterpret_cast<const uint32_t*>(sb + j * 32 * S::SPITCH + d * 4) >> 8 * lhalf;
        static_for<0, 2>([&](auto kc) {
            constexpr int kk = decltype(kc)::value;
            v4i fa[TI], fb[TJ];
            const uint32_t col = S::column(lrow, 4 * d + 2 * kk + lhalf);
#pragma unroll
            for (int i = 0; i < TI; ++i) fa[i] = *reinterpret_cast<const v4i*>(pa + i * 32 * S::PITCH + col);
#pragma unroll
            for (int j = 0; j < TJ; ++j) fb[j] = *reinterpret_cast<const v4i*>(pb + j * 32 * S::PITCH + col);
#pragma unroll
            for (int i = 0; i < TI; ++i) {
                const v8i xa = v8i{fa[i].x, fa[i].y, fa[i].z, fa[i].w, 0, 0, 0, 0};
#pragma unroll
                for (int j = 0; j < TJ; ++j) {
                    const v8i xb = v8i{fb[j].x, fb[j].y, fb[j].z, fb[j].w, 0, 0, 0, 0};
                    // first operand = n side, second = m side: a lane ends up with one m and runs of 4 n
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                        xb, xa, acc[i][j], 4, 4, 2 * kk, (int)ub[j], 2 * kk, (int)ua[i]);
                }
            }
        });
    });
}

// Whether the tile kernels store the output with the nontemporal hint: a final one (see store16) whose rows are whole sectors of
// 64 bytes.  In other rows a wave's piece of a row begins and ends inside a sector that the next tile completes; with the hint
// both parts go to memory by themselves, and more so the closer the stores follow each other.  Hint / no hint, in us:
// 25216 x 2808 x 96 bf16 69.8 / 29.6, 12608 x 1000 x 192 bf16 13.9 / 12.6, 36486 x 3180 x 320 FP32 169 / 112, 42568 x 684 x 384
// FP32 47.7 / 28.9.  Outputs of less than 24 MB, which the L2 caches hold either way, are even (4965 x 472 x 672 FP32 8.9 / 9.2, 5181
// x 1296 x 352 bf16 9.1 / 9.7), and whole sectors lose without the hint beyond the last-level cache (FP32, 256 MB: 1.07 to 1.2).
// (Computed from what the output stage needs anyway: one more kernel argument would be one more load that it waits for.)
__device__ __forceinline__ bool stream_output(const GemmArgs& g)
{
    if (g.split_k != 1) return false;
    const uint64_t pitch = (uint64_t)g.ldc * (g.c_bf16 ? 2u : 4u);
    return ((reinterpret_cast<uintptr_t>(g.c) | pitch) & 63u) == 0 || pitch * g.m < (24u << 20);
}

template <typename S, bool GELUQ>
__device__ __forceinline__ void gemm_tile(const GemmArgs& g, const uint32_t block, uint8_t* lds)
{
    constexpr int BM = S::BM, BN = S::BN, KS = S::KS;
    constexpr int CPR = S::ROWB / 16;                              // 16-byte chunks per row and step
    constexpr int A_CHUNKS = BM * CPR / T_NT, B_CHUNKS = BN * CPR / T_NT;
    constexpr int DPR = KS / 128;                                  // scale dwords per row and step
    constexpr int SDW = (BM + BN) * DPR, SC = (SDW + T_NT - 1) / T_NT;
    constexpr int TI = BM / 64, TJ = BN / 64;                      // MFMA tiles of a wave
    static_assert(BM * CPR % T_NT == 0 && BN * CPR % T_NT == 0, "tile/thread mismatch");

    uint32_t zsplit, tm, tn;
    decode_tile(g, block, zsplit, tm, tn);
    const uint32_t m0 = tm * BM, n0 = tn * BN;
    const uint32_t kbeg = zsplit * g.k_per_split;
    const uint32_t kend = min(g.k, kbeg + g.k_per_split);
    const uint32_t kbytes = g.k >> 1, kgroups = g.k >> 5;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const uint32_t lrow = lane & 31, lhalf = lane >> 5;

    // Rows past the matrix edge read the last valid row (their products are never stored).  Offsets fit 32 bits:
    // k <= 2^24, at most 128 rows.
    const uint8_t* a_base = g.a_codes + (size_t)m0 * kbytes;
    const uint8_t* b_base = g.b_codes + (size_t)n0 * kbytes;
    uint32_t a_off[A_CHUNKS], b_off[B_CHUNKS], s_left[SC];
    const uint8_t* s_src[SC];
    // chunk u of a thread: 16-byte column and row (where T_NT is a multiple of CPR: the same column in every row)
    auto ch = [&](int u) -> uint32_t { return (uint32_t)(tid + u * T_NT) % CPR; };
    const uint32_t mlast = g.m - 1 - m0, nlast = g.n - 1 - n0;
#pragma unroll
    for (int u = 0; u < A_CHUNKS; ++u) a_off[u] = min((uint32_t)(tid + u * T_NT) / CPR, mlast) * kbytes + ch(u) * 16;
#pragma unroll
    for (int u = 0; u < B_CHUNKS; ++u) b_off[u] = min((uint32_t)(tid + u * T_NT) / CPR, nlast) * kbytes + ch(u) * 16;
#pragma unroll
    for (int u = 0; u < SC; ++u) {
        const uint32_t row = min(tid + u * T_NT, SDW - 1) / DPR;
        const bool is_a = row < BM;
        const uint32_t lim = is_a ? g.m : g.n, r = is_a ? m0 + min(row, mlast) : n0 + min(row - BM, nlast);
        s_src[u] = (is_a ? g.a_scales : g.b_scales) + (size_t)r * kgroups;
        const uint64_t left = (uint64_t)(lim - r) * kgroups;
        s_left[u] = left < 0xFFFFFFFFull ? (uint32_t)left : 0xFFFFFFFFu;
    }

    v4i ra[A_CHUNKS], rb[B_CHUNKS];
    uint32_t rs[SC];
    auto gload = [&](uint32_t k0) {
        auto ok = [&](int u) { return k0 + ch(u) * 32 < kend; };
        const v4i z = v4i{0, 0, 0, 0};
        const uint8_t *pa = a_base + (k0 >> 1), *pb = b_base + (k0 >> 1);
#pragma unroll
        for (int u = 0; u < A_CHUNKS; ++u) ra[u] = ok(u) ? *reinterpret_cast<const v4i*>(pa + a_off[u]) : z;
#pragma unroll
        for (int u = 0; u < B_CHUNKS; ++u) rb[u] = ok(u) ? *reinterpret_cast<const v4i*>(pb + b_off[u]) : z;
#pragma unroll
        for (int u = 0; u < SC; ++u) {
            const uint32_t k = k0 + (tid + u * T_NT) % DPR * 128;
            rs[u] = k < kend && tid + u * T_NT < SDW ? load_scales4(s_src[u], k >> 5, s_left[u]) : 0u;
        }
    };
    auto lstore = [&](uint8_t* st) {
#pragma unroll
        for (int u = 0; u < A_CHUNKS; ++u) {
            const uint32_t row = (tid + u * T_NT) / CPR;
            *reinterpret_cast<v4i*>(st + row * S::PITCH + S::column(row, ch(u))) = ra[u];
        }
#pragma unroll
        for (int u = 0; u < B_CHUNKS; ++u) {
            const uint32_t row = (tid + u * T_NT) / CPR;
            *reinterpret_cast<v4i*>(st + (BM + row) * S::PITCH + S::column(row, ch(u))) = rb[u];
        }
#pragma unroll
        for (int u = 0; u < SC; ++u)
            if (tid + u * T_NT < SDW) *reinterpret_cast<uint32_t*>(st + (BM + BN) * S::PITCH + (tid + u * T_NT) / DPR * S::SPITCH + (tid + u * T_NT) % DPR * 4) = rs[u];
    };

    v16f acc[TI][TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    gload(kbeg);
    lstore(lds);
    __syncthreads();
    uint32_t cur = 0;
    for (uint32_t k0 = kbeg; k0 < kend; k0 += KS) {
        const bool more = S::STAGES > 1 && k0 + KS < kend;
        if (more) gload(k0 + KS);
        tile_multiply<S>(lds + cur, kend - k0, acc, wm, wn, lrow, lhalf);
        if (S::STAGES > 1) cur = cur ? 0u : (uint32_t)S::STAGE;
        if (more) lstore(lds + cur);
        __syncthreads();
    }
    // (the last barrier: every wave is done reading the stage buffers, which the output strips reuse)
    uint8_t* ep = lds + wave * 32 * S::EP_PITCH;
    if constexpr (GELUQ) {                                         // no K split
        static_assert(32 * TI * (16 * TJ + 16) + 32 * TI * TJ <= 32 * S::EP_PITCH, "strip");
        if (stream_output(g)) tile_epilogue<TI, TJ, true>(g, ep, acc, m0 + wm * (BM / 2), n0 + wn * (BN / 2), zsplit);
        else          tile_epilogue<TI, TJ, false>(g, ep, acc, m0 + wm * (BM / 2), n0 + wn * (BN / 2), zsplit);
        if (g.q_floor) tile_gelu_quant<true, TI, TJ>(g, ep, acc, m0 + wm * (BM / 2), n0 + wn * (BN / 2));
        else           tile_gelu_quant<false, TI, TJ>(g, ep, acc, m0 + wm * (BM / 2), n0 + wn * (BN / 2));
        return;
    }
    if (stream_output(g)) tile_epilogue<TI, TJ, true>(g, ep, acc, m0 + wm * (BM / 2), n0 + wn * (BN / 2), zsplit);
    else          tile_epilogue<TI, TJ, false>(g, ep, acc, m0 + wm * (BM / 2), n0 + wn * (BN / 2), zsplit);
}

using Tile128 = TileShape<128, 128, 128, 3>;
using Tile128x64 = TileShape<128, 64, 256, 3>;
using Tile64 = TileShape<64, 64, 512, 2>;
using Tile128Short = TileShape<128, 128, 384, 3>;

template <typename S, bool GELUQ = false>
__global__ __launch_bounds__(T_NT, S::OCC) void mx_gemm_tile_kernel(GemmArgs g)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[S::LDS];
    gemm_tile<S, GELUQ>(g, blockIdx.x, lds);
}

// Two products side by side: see launch_gemm_pair.  Workgroups from blocks0 (a multiple of 8) on work on the second.
template <typename S0, typename S1>
__global__ __launch_bounds__(T_NT, S0::OCC < S1::OCC ? S0::OCC : S1::OCC) void mx_gemm_tile_pair_kernel(GemmArgs g0, GemmArgs g1, uint32_t blocks0)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[S0::LDS > S1::LDS ? S0::LDS : S1::LDS];
    if (blockIdx.x >= blocks0)                                                               gemm_tile<S1, false>(g1, blockIdx.x - blocks0, lds);
    else if (blockIdx.x < g0.tiles_m * g0.tiles_n * (uint32_t)g0.split_k)                    gemm_tile<S0, false>(g0, blockIdx.x, lds);
}

// Y = Q1(X) Q2(W)^T + bias of a small layer where nothing else needs the codes (a forward pass without gradients), in one
// launch: each workgroup quantizes the 64 rows of X and of W that its tile needs straight into the LDS stages, 256 columns at
// a time, with the next step's sources in flight.  Rows are quantized once per tile that needs them, which costs less than
// the launch, the codes' way through memory and the wait between two kernels as long as there are few tiles and K is short
// (the rule stands at linear_fits_one_launch).  The codes, and the order of every sum, are those of the separate kernels.
struct QuantizedLinearArgs {
    const void* x;
    const void* w;
    const void* bias;          // n values or null
    int bias_bf16;
    GemmArgs g;                // sizes and output
};

constexpr int QL_NT = 512;     // eight waves quantize, the first four multiply

template <typename XT, typename WT, bool FLOOR>
__global__ __launch_bounds__(QL_NT, 2) void mx_quantized_linear_kernel(QuantizedLinearArgs a)
{
    using S = TileShape<64, 64, 256, 2>;
    constexpr int CPR = S::KS / 8, RPP = QL_NT / CPR, ROWS = 64 / RPP;      // 8-element chunks per row, rows per pass, passes
    __shared__ __attribute__((aligned(16))) uint8_t lds[S::LDS];
    const GemmArgs& g = a.g;
    uint32_t zsplit, tm, tn;
    decode_tile(g, blockIdx.x, zsplit, tm, tn);
    const uint32_t m0 = tm * 64, n0 = tn * 64, k = g.k;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave >> 1) & 1, wn = wave & 1;
    const uint32_t lrow = lane & 31, lhalf = lane >> 5;
    const uint32_t c = tid % CPR, r0 = tid / CPR;
    const uint32_t mlast = g.m - 1 - m0, nlast = g.n - 1 - n0;
    const XT* x = static_cast<const XT*>(a.x) + (size_t)m0 * k;
    const WT* w = static_cast<const WT*>(a.w) + (size_t)n0 * k;

    mxd::Raw8<XT> xr[ROWS];
    mxd::Raw8<WT> wr[ROWS];
    auto load = [&](uint32_t k0) {
        const uint32_t col = k0 + c * 8;                                   // whole groups lie inside or past K
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            xr[u] = mxd::Raw8<XT>{};
            wr[u] = mxd::Raw8<WT>{};
            if (col < k) {
                xr[u] = mxd::load_raw8_shared(x + (size_t)min(r0 + u * RPP, mlast) * k + col);
                wr[u] = mxd::load_raw8_shared(w + (size_t)min(r0 + u * RPP, nlast) * k + col);
            }
        }
    };
    auto encode = [&](uint8_t* st) {
        auto put = [&](const auto& raw, uint32_t row) {
            const uint32_t byte = mxd::row_scale_byte<FLOOR>(raw);
            *reinterpret_cast<uint32_t*>(st + row * S::PITCH + S::column(row, c >> 2) + (c & 3) * 4) = mxd::rtn_codes8(raw, byte);
            if ((c & 3) == 0) st[128 * S::PITCH + row * S::SPITCH + (c >> 2)] = (uint8_t)byte;
        };
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            put(xr[u], r0 + u * RPP);
            put(wr[u], 64 + r0 + u * RPP);
        }
    };

    v16f acc[1][1];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][0][r] = 0.f;
    load(0);
    encode(lds);
    __syncthreads();
    uint32_t cur = 0;
    for (uint32_t k0 = 0; k0 < k; k0 += S::KS) {
        const bool more = k0 + S::KS < k;
        if (more) load(k0 + S::KS);
        if (wave < 4) tile_multiply<S>(lds + cur, k - k0, acc, wm, wn, lrow, lhalf);
        cur = cur ? 0u : (uint32_t)S::STAGE;
        if (more) encode(lds + cur);
        __syncthreads();
    }
    if (wave >= 4) return;
    const uint32_t nbase = n0 + wn * 32;
    if (a.bias != nullptr && nbase < g.n) {                                // n % 32 == 0
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t col = nbase + 8 * q + 4 * lhalf;
            if (a.bias_bf16) {
                const uint2 v = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(a.bias) + col);
                acc[0][0][4 * q] += __uint_as_float(v.x << 16);     acc[0][0][4 * q + 1] += __uint_as_float(v.x & 0xFFFF0000u);
                acc[0][0][4 * q + 2] += __uint_as_float(v.y << 16); acc[0][0][4 * q + 3] += __uint_as_float(v.y & 0xFFFF0000u);
            } else {
                const v4f v = *reinterpret_cast<const v4f*>(static_cast<const float*>(a.bias) + col);
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[0][0][4 * q + r] += v[r];
            }
        }
    }
    tile_epilogue<1, 1, true>(g, lds + wave * 32 * S::EP_PITCH, acc, m0 + wm * 32, nbase, 0);
}

// Sum the split-K partials in a fixed order and write the final output.
// The first `tail_blocks` workgroups finish a column sum, which saves that its own launch: few and each a chain of loads,
// they run beside the reduction when they start with it.  4096 x 1024, four splits, 197 blocks of column sums: 25.6 us with
// them as the last workgroups and one load at a time, 15.8 now, 14.4 without column sums.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* part, int split, uint32_t m, uint32_t n,
                                     void* c, int64_t ldc, int c_bf16, const float* bias, mxl::ColumnSumTail tail, uint32_t tail_blocks)
{
    if (blockIdx.x < tail_blocks) {
        mxl::column_sum_finish(tail, blockIdx.x);
        return;
    }
    const uint32_t block = blockIdx.x - tail_blocks;
    size_t idx = (size_t)block * blockDim.x + threadIdx.x;
    size_t total = (size_t)m * n;
    if (idx >= total) return;
    float s = 0.f;
    for (int z = 0; z < split; ++z) s += part[(size_t)z * total + idx];
    uint32_t r = (uint32_t)(idx / n), col = (uint32_t)(idx - (size_t)r * n);
    if (bias) s += bias[col];
    if (c_bf16) static_cast<uint16_t*>(c)[(size_t)r * ldc + col] = f32_to_bf16_rne(s);
    else        static_cast<float*>(c)[(size_t)r * ldc + col] = s;
}

// The same for n % 4 == 0 and 16-byte aligned rows of the output: four columns per thread, the
// partial loads of a thread issued back to back (same summation order per element).
__global__ __launch_bounds__(256) void splitk_reduce4_kernel(const float* part, int split, uint32_t m, uint32_t n,
                                      void* c, int64_t ldc, int c_bf16, const float* bias, mxl::ColumnSumTail tail, uint32_t tail_blocks)
{
    if (blockIdx.x < tail_blocks) {
        mxl::column_sum_finish(tail, blockIdx.x);
        return;
    }
    const uint32_t block = blockIdx.x - tail_blocks;
    const size_t q = (size_t)block * blockDim.x + threadIdx.x;            // index of a group of 4 columns
    const size_t total = (size_t)m * n;
    if (q * 4 >= total) return;
    const float4* p4 = reinterpret_cast<const float4*>(part) + q;
    const size_t zstride = total / 4;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    int z = 0;
    for (; z + 4 <= split; z += 4) {
        const float4 a = p4[(size_t)z * zstride], b = p4[(size_t)(z + 1) * zstride];
        const float4 d = p4[(size_t)(z + 2) * zstride], e = p4[(size_t)(z + 3) * zstride];
        s.x = (((s.x + a.x) + b.x) + d.x) + e.x;
        s.y = (((s.y + a.y) + b.y) + d.y) + e.y;
        s.z = (((s.z + a.z) + b.z) + d.z) + e.z;
        s.w = (((s.w + a.w) + b.w) + d.w) + e.w;
    }
    for (; z < split; ++z) {
        const float4 a = p4[(size_t)z * zstride];
        s.x += a.x; s.y += a.y; s.z += a.z; s.w += a.w;
    }
    const size_t idx = q * 4;
    const uint32_t r = (uint32_t)(idx / n), col = (uint32_t)(idx - (size_t)r * n);
    if (bias) {
        const float4 bv = *reinterpret_cast<const float4*>(bias + col);
        s.x += bv.x; s.y += bv.y; s.z += bv.z; s.w += bv.w;
    }
    if (c_bf16) {
        uint2 o;
        o.x = f32x2_to_bf16x2(s.x, s.y);
        o.y = f32x2_to_bf16x2(s.z, s.w);
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(c) + (size_t)r * ldc + col) = o;
    } else {
        *reinterpret_cast<float4*>(static_cast<float*>(c) + (size_t)r * ldc + col) = s;
    }
}

// ---------------------------------------------------------------------------
// Helpers of the main path (K range of at least 512 per split; mx_gemm_pingpong_kernel below).
// ---------------------------------------------------------------------------

// No instruction is scheduled across this point.
#define MX_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

constexpr int P_EP_PITCH = 144;                              // output staging: 128 bytes of payload per row, padded
constexpr int P_EP_BYTES = 32 * P_EP_PITCH;                  // per wave

// Lane index within the wave, computed anew at each use (two VALU instructions): code that
// needs lane-derived values once per tile does not hold registers for them across the K loop.
__device__ __forceinline__ uint32_t fresh_lane_id()
{
    uint32_t l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}

// Accumulators of one wave (64 rows x 128 columns) -> global through a 32-row LDS strip
// holding 128 bytes per row: 64 bf16 or 32 fp32 columns at a time.  A store instruction
// of the wave covers 8 whole 128-byte row segments.
typedef int v2i __attribute__((ext_vector_type(2)));

// The same output stage for a wave tile that lies wholly inside the matrix and whose rows can be
// stored 16 bytes at a time (the common case; every tile of a ViT-B product): no bounds tests, no
// per-store address arithmetic (a store's address is a uniform tile pointer plus one per-lane
// offset that is computed once), and no waits between the LDS writes and reads of a chunk (the LDS
// executes a wave's instructions in order; the compiler waits where a register needs its data).
// The compiler keeps the strip's accesses in program order because writes and reads go through
// pointers into the same array whose lane offsets it cannot tell apart; strip_order() between them
// says so, and costs this kernel 1 % at long K (50432 x 768 x 3072 72.6 us, 73.2 with it).
// BIAS: add the 128 FP32 bias values at LDS address `bias` (column nbase first).
template <bool STREAM, bool BIAS>
__device__ __forceinline__ void gemm_epilogue_interior(const GemmArgs& g, lds_u8* ep, v16f (&acc)[2][4],
                                                       uint32_t mrow0, uint32_t nbase, uint32_t zsplit, int64_t ldc,
                                                       const lds_u8* bias)
{
    typedef __attribute__((address_space(3))) v4i lds_v4i;
    typedef __attribute__((address_space(3))) v2i lds_v2i;
    typedef __attribute__((address_space(3))) v4f lds_v4f;
    const uint32_t lane = fresh_lane_id();
    const uint32_t lrow = lane & 31, lhalf = lane >> 5;
    const uint32_t rrow = lane >> 3, rchunk = lane & 7;
    const lds_u8* rd = ep + rrow * P_EP_PITCH + rchunk * 16;
    auto bias4 = [&](int jb, int q) -> v4f {
        return *reinterpret_cast<const lds_v4f*>(bias + (32 * jb + 8 * q + 4 * lhalf) * 4);
    };
    // Four (bf16) or eight (FP32) chunks of 32 rows x 128 bytes pass through the wave's LDS strip.  The
    // strip's accesses execute in program order, so the writes of chunk c+1 are issued right after the
    // reads of chunk c and before the global stores that wait for those reads: the LDS round trip of a
    // chunk is hidden behind the next chunk's conversion instead of being waited for 16 times.
    if (g.c_bf16 && g.split_k == 1) {
        lds_u8* wr = ep + lrow * P_EP_PITCH + lhalf * 8;
        uint8_t* tile = static_cast<uint8_t*>(g.c) + ((size_t)mrow0 * ldc + nbase) * 2;       // uniform
        const uint32_t voff = rrow * (uint32_t)ldc * 2u + rchunk * 16u;
        auto write_chunk = [&](int i, int jp) {
#pragma unroll
            for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const v16f& a = acc[i][2 * jp + jj];
                    v2i pk;
                    if (BIAS) {
                        const v4f bv = bias4(2 * jp + jj, q);
                        pk.x = (int)f32x2_to_bf16x2(a[4 * q] + bv.x, a[4 * q + 1] + bv.y);
                        pk.y = (int)f32x2_to_bf16x2(a[4 * q + 2] + bv.z, a[4 * q + 3] + bv.w);
                    } else {
                        pk.x = (int)f32x2_to_bf16x2(a[4 * q], a[4 * q + 1]);
                        pk.y = (int)f32x2_to_bf16x2(a[4 * q + 2], a[4 * q + 3]);
                    }
                    *reinterpret_cast<lds_v2i*>(wr + (32 * jj + 8 * q) * 2) = pk;
                }
        };
        v4i v[4];
        write_chunk(0, 0);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int i = c >> 1, jp = c & 1;
#pragma unroll
            for (int it = 0; it < 4; ++it) v[it] = *reinterpret_cast<const lds_v4i*>(rd + it * 8 * P_EP_PITCH);
            if (c + 1 < 4) write_chunk((c + 1) >> 1, (c + 1) & 1);
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                uint8_t* dst = tile + ((size_t)(i * 32 + it * 8) * ldc + jp * 64) * 2;            // uniform
                store16<STREAM>(dst + voff, v[it]);
            }
        }
    } else {
        lds_u8* wr = ep + lrow * P_EP_PITCH + lhalf * 16;
        float* base = static_cast<float*>(g.c);
        if (g.split_k > 1) base += (size_t)zsplit * g.m * g.n;
        uint8_t* tile = reinterpret_cast<uint8_t*>(base) + ((size_t)mrow0 * ldc + nbase) * 4;
        const uint32_t voff = rrow * (uint32_t)ldc * 4u + rchunk * 16u;
        auto write_chunk = [&](int i, int j) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v4f o = v4f{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                if (BIAS) o += bias4(j, q);
                *reinterpret_cast<lds_v4f*>(wr + 8 * q * 4) = o;
            }
        };
        v4i v[4];
        write_chunk(0, 0);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int i = c >> 2, j = c & 3;
#pragma unroll
            for (int it = 0; it < 4; ++it) v[it] = *reinterpret_cast<const lds_v4i*>(rd + it * 8 * P_EP_PITCH);
            if (c + 1 < 8) write_chunk((c + 1) >> 2, (c + 1) & 3);
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                uint8_t* dst = tile + ((size_t)(i * 32 + it * 8) * ldc + j * 32) * 4;             // uniform
                store16<STREAM>(dst + voff, v[it]);
            }
        }
    }
}

// Second output stage of the fused forward product of an MLP's first layer: the next layer's forward
// quantizer Q(1) (Eq. 3; 1x32 groups along the output columns, which are the next layer's contraction
// dimension, round_D) applied to GELU(product + bias), from the FP32 accumulators.  Runs after the stage
// that stores the pre-activation and reuses the wave's LDS strip.
// A lane holds, of each 32 x 32 MFMA tile (i, j), 16 of the 32 columns of one row: the four runs
// 8q + 4 * lhalf + (0..3); the other 16 are in the lane 32 away.  Group maximum: the lane's 16 values, then one
// exchange with that lane.  The 16 codes of a lane are four 2-byte pieces of the group's 16 bytes; they go to
// the strip ([64 rows][64 B] codes, then [64 rows][4] scale bytes) and leave as 16-byte pieces, 64 contiguous
// bytes per row.  Rows beyond m and column groups beyond n (n % 32 == 0) are not stored.
template <bool FLOOR>
__device__ __forceinline__ void gemm_epilogue_gelu_quant(const GemmArgs& g, lds_u8* ep, v16f (&acc)[2][4],
                                                         uint32_t mrow0, uint32_t nbase, const lds_u8* bias)
{
    typedef __attribute__((address_space(3))) v4f lds_v4f;
    typedef __attribute__((address_space(3))) v4i lds_v4i;
    typedef __attribute__((address_space(3))) uint16_t lds_u16;
    typedef __attribute__((address_space(3))) uint32_t lds_u32;
    const uint32_t lane = fresh_lane_id();
    const uint32_t lrow = lane & 31, lhalf = lane >> 5;
    lds_u8* scale_strip = ep + 4096;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float v[16];
            uint32_t m = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v4f bv = *reinterpret_cast<const lds_v4f*>(bias + (32 * j + 8 * q + 4 * lhalf) * 4);
                const float pre[4] = {acc[i][j][4 * q] + bv.x, acc[i][j][4 * q + 1] + bv.y, acc[i][j][4 * q + 2] + bv.z,
                                      acc[i][j][4 * q + 3] + bv.w};
                float post[4];
                gelu4_f32(pre, post);
#pragma unroll
                for (int r = 0; r < 4; ++r) v[4 * q + r] = post[r];
                m = mxd::absmax3_bits(v[4 * q], v[4 * q + 1], m);
                m = mxd::absmax3_bits(v[4 * q + 2], v[4 * q + 3], m);
            }
            const auto sw = __builtin_amdgcn_permlane32_swap(m, m, false, false);
            m = sw[0] > sw[1] ? sw[0] : sw[1];
            const uint32_t byte = mxd::scale_byte(m, FLOOR);
            const float scale = mxd::scale_operand(byte);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t pk = mxd::cvt_rtn_f32<0>(0u, v[4 * q], v[4 * q + 1], scale);
                pk = mxd::cvt_rtn_f32<1>(pk, v[4 * q + 2], v[4 * q + 3], scale);
                *reinterpret_cast<lds_u16*>(ep + (i * 32 + lrow) * 64 + 16 * j + 4 * q + 2 * lhalf) = (uint16_t)pk;
            }
            if (lhalf == 0) scale_strip[(i * 32 + lrow) * 4 + j] = (uint8_t)byte;
        }
    asm volatile("" ::: "memory");          // the strip is read back below through other lanes' addresses
    // codes: 4 lanes per row (one column group each), 16 rows per instruction
    const uint32_t half_n = g.n >> 1, grp_n = g.n >> 5;
    const uint32_t piece = lane & 3, prow = lane >> 2;
    const bool group_ok = nbase + 32 * piece < g.n;
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const uint32_t row = it * 16 + prow;
        const v4i c = *reinterpret_cast<const lds_v4i*>(ep + row * 64 + piece * 16);
        if (group_ok && mrow0 + row < g.m)
            *reinterpret_cast<v4i*>(g.q_codes + (size_t)(mrow0 + row) * half_n + (nbase >> 1) + piece * 16) = c;
    }
    // scale bytes: one row per lane
    {
        const uint32_t sc = *reinterpret_cast<const lds_u32*>(scale_strip + lane * 4);
        if (mrow0 + lane < g.m) {
            uint8_t* dst = g.q_scales + (size_t)(mrow0 + lane) * grp_n + (nbase >> 5);
            if (nbase + 128 <= g.n && (grp_n & 3u) == 0u && (reinterpret_cast<uintptr_t>(g.q_scales) & 3u) == 0u) {
                *reinterpret_cast<uint32_t*>(dst) = sc;
            } else {
                for (uint32_t b = 0; b < 4; ++b)
                    if (nbase + 32 * b < g.n) dst[b] = (uint8_t)(sc >> (8 * b));
            }
        }
    }
}

// bias: LDS address of the bias value of column nbase (FP32, 128 values), or null.
template <bool STREAM>
__device__ __forceinline__ void gemm_epilogue_chunked(const GemmArgs& g, uint8_t* ep, v16f (&acc)[2][4],
                                                      uint32_t mrow0, uint32_t nbase, int lane_in, uint32_t zsplit,
                                                      const __attribute__((address_space(3))) uint8_t* bias)
{
    // bias of the four columns a lane holds in accumulator registers 4q..4q+3 of column block jb
    auto bias4 = [&](int jb, int q, uint32_t lhalf) -> v4f {
        if (bias == nullptr) return v4f{0.f, 0.f, 0.f, 0.f};
        return *reinterpret_cast<const __attribute__((address_space(3))) v4f*>(bias + (32 * jb + 8 * q + 4 * lhalf) * 4);
    };
    // lane-derived indices are recomputed at every call instead of living across the K loop
    (void)lane_in;
    const uint32_t lane = fresh_lane_id();
    const uint32_t lrow = lane & 31, lhalf = lane >> 5;
    const uint32_t rrow = lane >> 3, rchunk = lane & 7;
    float* cf = static_cast<float*>(g.c);
    uint16_t* ch = static_cast<uint16_t*>(g.c);
    int64_t ldc = g.ldc;
    if (g.split_k > 1) {
        cf += (size_t)zsplit * g.m * g.n;
        ldc = g.n;
    }
    const bool as_bf16 = g.c_bf16 && g.split_k == 1;
    if (as_bf16) {
        const bool vec_ok = (ldc & 7) == 0 && (reinterpret_cast<uintptr_t>(ch) & 15) == 0;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int jp = 0; jp < 2; ++jp) {
#pragma unroll
                for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const v16f& a = acc[i][2 * jp + jj];
                        const v4f bv = bias4(2 * jp + jj, q, lhalf);
                        uint2 pk;
                        pk.x = f32x2_to_bf16x2(a[4 * q] + bv.x, a[4 * q + 1] + bv.y);
                        pk.y = f32x2_to_bf16x2(a[4 * q + 2] + bv.z, a[4 * q + 3] + bv.w);
                        *reinterpret_cast<uint2*>(ep + lrow * P_EP_PITCH + (32 * jj + 8 * q + 4 * lhalf) * 2) = pk;
                    }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
                for (int it = 0; it < 4; ++it) {
                    const uint32_t row = it * 8 + rrow;
                    const uint32_t mm = mrow0 + i * 32 + row, nn = nbase + jp * 64 + rchunk * 8;
                    uint4 v = *reinterpret_cast<const uint4*>(ep + row * P_EP_PITCH + rchunk * 16);
                    if (mm < g.m && nn < g.n) {
                        uint16_t* dst = ch + (size_t)mm * ldc + nn;
                        if (nn + 8 <= g.n && vec_ok) {
                            store16<STREAM>(dst, v4i{(int)v.x, (int)v.y, (int)v.z, (int)v.w});
                        } else {
                            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
                            for (int e = 0; e < 8; ++e)
                                if (nn + e < g.n) dst[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
                        }
                    }
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
    } else {
        const bool vec_ok = (ldc & 3) == 0 && (reinterpret_cast<uintptr_t>(cf) & 15) == 0;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const v4f bv = bias4(j, q, lhalf);
                    *reinterpret_cast<float4*>(ep + lrow * P_EP_PITCH + (8 * q + 4 * lhalf) * 4) =
                        make_float4(acc[i][j][4 * q] + bv.x, acc[i][j][4 * q + 1] + bv.y, acc[i][j][4 * q + 2] + bv.z,
                                    acc[i][j][4 * q + 3] + bv.w);
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
                for (int it = 0; it < 4; ++it) {
                    const uint32_t row = it * 8 + rrow;
                    const uint32_t mm = mrow0 + i * 32 + row, nn = nbase + j * 32 + rchunk * 4;
                    float4 v = *reinterpret_cast<const float4*>(ep + row * P_EP_PITCH + rchunk * 16);
                    if (mm < g.m && nn < g.n) {
                        float* dst = cf + (size_t)mm * ldc + nn;
                        if (nn + 4 <= g.n && vec_ok) {
                            store16<STREAM>(dst, v4i{__float_as_int(v.x), __float_as_int(v.y), __float_as_int(v.z), __float_as_int(v.w)});
                        } else {
                            const float w[4] = {v.x, v.y, v.z, v.w};
                            for (int e = 0; e < 4; ++e)
                                if (nn + e < g.n) dst[e] = w[e];
                        }
                    }
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
    }
}

// ---------------------------------------------------------------------------
// Ping-pong form of the main path: one workgroup of 8 waves per CU, tile 256 x 256.
// Waves 0-3 (group 0) and 4-7 (group 1) own the left and right 128 columns; wave w and
// wave w+4 sit on the same SIMD.  Time is cut into slots separated by workgroup barriers.
// In every slot one group issues its 16 MFMAs of a K step (M phase) while the other group
// reads the operands of its next K step from LDS and issues DMA loads (L phase); then they
// swap.  The matrix pipe of a SIMD always has exactly one wave feeding it, and no LDS or
// DMA latency sits between two MFMA bursts of the same wave.
//   Per 256 x 256 x 128 step the CU loads 32 KB through L2 -> LDS instead of the 2 x 24 KB of
//   two 256 x 128 workgroups.
//   LDS: 3 code stages x 32 KB | 3 scale slots x [512 rows][16 B] | output staging 8 x 4.5 KB |
//        2 x 1 KB of bias values (the tile being multiplied and the one being loaded).
// Two cursors run over the workgroup's tile list.  The read cursor names the K step whose
// operands the next L phase reads; the issue cursor runs two stages ahead of it (also across
// tile boundaries) and names the stage the same L phase loads.  Stage q of a tile lives in
// buffer (global stage count) % 3, scale block j in slot (global block count) % 3.
// Safety of the ring: the L phase of step s reads stage s and overwrites the buffer of stage
// s-1, whose last readers (the other group's L phase of step s-1, and this group's) finished
// before the previous barrier.  Each wave ends an L phase with a wait for all loads it issued
// in earlier phases, so stage s+1 is complete, and visible after the barrier, before its first
// reader.  Scale block j of a tile is issued with stage 4j-1 (block 0 with stage 0), at least
// two steps before its first reader and after the last reader of the slot's previous block.
// ---------------------------------------------------------------------------
constexpr int Q_BM = 256, Q_BN = 256, Q_NT = 512, Q_WAVES = 8, Q_STAGES = 3;
constexpr int Q_STAGE_BYTES = (Q_BM + Q_BN) * 64;                       // 32768
constexpr int Q_SCALE_OFF = Q_STAGES * Q_STAGE_BYTES;                   // 98304
constexpr int Q_SCALE_SLOT = (Q_BM + Q_BN) * 16;                        // 8192
constexpr int Q_EP_OFF = Q_SCALE_OFF + 3 * Q_SCALE_SLOT;                // 122880
constexpr int Q_BIAS_OFF = Q_EP_OFF + Q_WAVES * P_EP_BYTES;             // 159744: two slots of 256 bias values
constexpr int Q_LDS_BYTES = Q_BIAS_OFF + 2 * 1024;                      // 161792
static_assert(Q_LDS_BYTES <= 160 * 1024, "one workgroup per CU");
constexpr unsigned Q_SLOTS = 256;

__device__ __forceinline__ void barrier_after_mfma(v16f (&acc)[2][4])
{
    // the accumulators pass through the statement: the MFMAs before it stay before it
    asm volatile("s_barrier"
                 : "+v"(acc[0][0]), "+v"(acc[0][1]), "+v"(acc[0][2]), "+v"(acc[0][3]),
                   "+v"(acc[1][0]), "+v"(acc[1][1]), "+v"(acc[1][2]), "+v"(acc[1][3])
                 :
                 : "memory");
}

// DMA load, 16 bytes per lane: lane i's bytes [base + voff, +16) land at LDS byte address
// lds_addr + 16 * i.  Written as an assembly statement for two reasons.  The compiler then keeps no
// record of outstanding loads into LDS: with the builtin it waits for all of them (vmcnt(0)) before
// the first LDS write that might overlap, which here is the output staging that runs while the
// next tile's loads are in flight; this kernel places every such wait itself.  And the address
// takes the scalar-base form directly (uniform 64-bit base, 32-bit lane offset) instead of 64-bit
// per-lane addresses.  M0 (the LDS destination) is listed as clobbered.
__device__ __forceinline__ void dma_load16_at(uint32_t lds_addr, const uint8_t* base, uint32_t voff)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds_addr), "v"(voff), "s"(base)
                 : "memory", "m0");
}

// The whole tile walk of one wave; GRP (0: columns 0-127, M phase first; 1: columns 128-255, L phase
// first) is a template parameter so that each group's loop is straight-line code.  All cursor
// state is wave-uniform (scalar registers) and advanced with compares and adds only.
template <int GRP, bool BIAS, bool GELUQ>
__device__ __forceinline__ void pingpong_wave(const GemmArgs& g, lds_u8* lds, const int wave)
{
    const uint32_t tiles = g.tiles_m * g.tiles_n, total = tiles * (uint32_t)g.split_k;
    const uint32_t xcd = blockIdx.x % 8, per = total / 8, rem = total % 8;
    const uint32_t range_end = (xcd + 1) * per + min(xcd + 1, rem);
    const uint32_t stride = (gridDim.x - xcd + 7) / 8;          // workgroups on this XCD
    const uint32_t first = xcd * per + min(xcd, rem) + blockIdx.x / 8;
    if (first >= range_end) return;

    MX_PROBE_INIT
    const uint32_t kbytes = g.k >> 1, kgroups = g.k >> 5;
    const int lane = threadIdx.x & 63;
    const int wm = wave & 3;
    const uint32_t lrow = lane & 31, lhalf = lane >> 5;
    const uint32_t swz = (lrow >> 2) & 3;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;

    // K steps per tile: the same for every tile but those of the last K split
    const int nk_full = (int)(g.k_per_split >> 7);
    const int nk_tail = (int)((g.k - (uint32_t)(g.split_k - 1) * g.k_per_split) >> 7);
    const uint32_t tail_first = tiles * (uint32_t)(g.split_k - 1);
    auto tile_steps = [&](uint32_t t) -> int { return t >= tail_first ? nk_tail : nk_full; };

    // ---- issue cursor: next stage to load.  The common path of a phase is straight-line
    //      scalar code; everything rare (a scale block is due, the tile ends) sits behind one
    //      branch each.  When the tile list is exhausted the cursor keeps re-loading the last
    //      stage (i_step = 0) into buffers that no longer have readers. ----
    uint32_t a_off[2], b_off[2], s_off;
    const uint8_t *a_ptr, *b_ptr, *s_base;
    uint32_t i_tile = first;
    int i_nk = 0, i_q = 0;              // K steps of the issue tile, next stage of it to load
    int i_due = 0, i_j = 0;             // stage that scale block i_j travels with
    uint32_t i_step = 64;               // bytes the code pointers advance per stage
    uint32_t i_dst = lds0 + wave * 2048;                          // this wave's A piece of the stage buffer
    uint32_t i_sdst = lds0 + Q_SCALE_OFF + wave * 1024;           // this wave's piece of the scale slot
    int i_buf = 0, i_slot = 0;
    uint32_t i_bias = lds0 + Q_BIAS_OFF;                          // bias slot of the next tile to be issued
    auto set_issue_tile = [&](uint32_t t) {
        const uint32_t z = t / tiles, r = t - z * tiles, tm = r / g.tiles_n;
        const uint32_t m0 = tm * Q_BM, n0 = (r - tm * g.tiles_n) * Q_BN;
        const uint32_t kbeg = z * g.k_per_split;
        const uint32_t mlast = g.m - 1 - m0, nlast = g.n - 1 - n0;
        a_ptr = g.a_codes + (size_t)m0 * kbytes + (kbeg >> 1);
        b_ptr = g.b_codes + (size_t)n0 * kbytes + (kbeg >> 1);
        const uint32_t ln = fresh_lane_id();
        const uint32_t lr = ln >> 2, lc = ((ln & 3) ^ ((ln >> 4) & 3)) << 4;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            a_off[u] = min(lr + (2 * wave + u) * 16, mlast) * kbytes + lc;
            b_off[u] = min(lr + (2 * wave + u) * 16, nlast) * kbytes + lc;
        }
        // scale rows: waves 0-3 fetch the A rows [64w, 64w+64), waves 4-7 the B rows [64(w-4), +64)
        if (GRP == 0) {
            s_base = g.a_scales + (size_t)m0 * kgroups + (kbeg >> 5);
            s_off = min((uint32_t)(wm * 64) + ln, mlast) * kgroups;
        } else {
            s_base = g.b_scales + (size_t)n0 * kgroups + (kbeg >> 5);
            s_off = min((uint32_t)(wm * 64) + ln, nlast) * kgroups;
        }
        i_nk = tile_steps(t);
        i_q = 0;
        i_due = 0;
        i_j = 0;
        // The tile's 256 bias values go to the slot that the tile before the previous one used; that tile's
        // output stage ended, in every wave, before the barriers of the previous tile's K loop (>= 4 steps),
        // and this point lies inside that loop.  One wave loads; its later waits cover the load (loads
        // complete in order) and barriers follow before any wave reads the slot.
        if (BIAS && GRP == 0 && wave == 0) {
            dma_load16_at(i_bias, reinterpret_cast<const uint8_t*>(g.bias + n0), min(4u * ln, g.n - 4u - n0) * 4u);
            i_bias = i_bias == lds0 + Q_BIAS_OFF ? i_bias + 1024u : i_bias - 1024u;
        }
    };
    // Loads the next stage (and the scale block that travels with it) and waits for every load
    // issued in earlier phases.
    auto issue_and_wait = [&]() {
        if (i_q == i_due) {                                      // once per 4 K steps
            const int off = min(4 * i_j, i_nk - 4) * 4;
            dma_load16_at(i_sdst, s_base + off, s_off);
            i_sdst += Q_SCALE_SLOT;
            if (++i_slot == 3) { i_slot = 0; i_sdst -= 3 * Q_SCALE_SLOT; }
            ++i_j;
            i_due = 4 * i_j < i_nk ? 4 * i_j - 1 : 0x7FFFFFFF;
            dma_load16_at(i_dst, a_ptr, a_off[0]);
            dma_load16_at(i_dst + 1024, a_ptr, a_off[1]);
            dma_load16_at(i_dst + Q_BM * 64, b_ptr, b_off[0]);
            dma_load16_at(i_dst + Q_BM * 64 + 1024, b_ptr, b_off[1]);
            MX_PROBE(1);
            asm volatile("s_waitcnt vmcnt(5)" ::: "memory");
        } else {
            dma_load16_at(i_dst, a_ptr, a_off[0]);
            dma_load16_at(i_dst + 1024, a_ptr, a_off[1]);
            dma_load16_at(i_dst + Q_BM * 64, b_ptr, b_off[0]);
            dma_load16_at(i_dst + Q_BM * 64 + 1024, b_ptr, b_off[1]);
            MX_PROBE(1);
            asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
        }
        MX_PROBE(2);
        a_ptr += i_step;
        b_ptr += i_step;
        i_dst = i_buf == 2 ? i_dst - 2 * Q_STAGE_BYTES : i_dst + Q_STAGE_BYTES;
        i_buf = i_buf == 2 ? 0 : i_buf + 1;
        if (++i_q == i_nk) {                                     // once per tile
            i_tile += stride;
            if (i_tile < range_end) {
                set_issue_tile(i_tile);
            } else {                                             // nothing left: stay on the last stage
                a_ptr -= 64;
                b_ptr -= 64;
                i_step = 0;
                i_q = 0;
                i_nk = 0x7FFFFFFF;
                i_due = -1;
            }
        }
    };

    // ---- read cursor: K step whose operands the next L phase reads (past the end of the tile
    //      list it keeps reading the buffers; those operands are never used) ----
    uint32_t r_tile = first;
    int r_nk = tile_steps(first), r_s = 0;
    int r_buf = 0, r_slot = 0;
    uint32_t r_src = 0;                 // byte offset of the stage buffer
    uint32_t r_sc = Q_SCALE_OFF;        // byte offset of this step's scale dwords: slot + 4 * (step within block)

    // per-lane parts of the LDS read addresses
    const uint32_t a_rd = (wm * 64 + lrow) * 64, b_rd = Q_BM * 64 + (GRP * 128 + lrow) * 64;
    const uint32_t a_rd0 = a_rd + (((0 + lhalf) ^ swz) << 4), a_rd1 = a_rd + (((2 + lhalf) ^ swz) << 4);
    const uint32_t b_rd0 = b_rd + (((0 + lhalf) ^ swz) << 4), b_rd1 = b_rd + (((2 + lhalf) ^ swz) << 4);
    const uint32_t sa_rd = (wm * 64 + lane) * 16, sb_rd = (Q_BM + GRP * 128 + lane) * 16;    // lane, not lane % 32

    struct Frag { v4i a[2]; v4i b[4]; };
    Frag f[2];
    uint32_t sca[2], scb[4];
    v16f acc[2][4];

    auto load_phase = [&]() {
        uint32_t va, vb0, vb1;
        MX_PROBE(0);
        {
            // scale dwords of this K step: one read serves two 32-row blocks (lanes 0-31 the first,
            // lanes 32-63 the second; the 16-byte row pitch makes each read a 4-way bank conflict
            // whether or not the two half waves read the same rows), then the halves are exchanged
            const lds_u8* sp = lds + r_sc;
            va = *reinterpret_cast<const __attribute__((address_space(3))) uint32_t*>(sp + sa_rd);
            vb0 = *reinterpret_cast<const __attribute__((address_space(3))) uint32_t*>(sp + sb_rd);
            vb1 = *reinterpret_cast<const __attribute__((address_space(3))) uint32_t*>(sp + sb_rd + 1024);
            const lds_u8* base = lds + r_src;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                f[0].a[i] = *reinterpret_cast<const __attribute__((address_space(3))) v4i*>(base + a_rd0 + i * 2048);
                f[1].a[i] = *reinterpret_cast<const __attribute__((address_space(3))) v4i*>(base + a_rd1 + i * 2048);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f[0].b[j] = *reinterpret_cast<const __attribute__((address_space(3))) v4i*>(base + b_rd0 + j * 2048);
                f[1].b[j] = *reinterpret_cast<const __attribute__((address_space(3))) v4i*>(base + b_rd1 + j * 2048);
            }
            // advance to the next K step
            r_src = r_buf == 2 ? 0 : r_src + Q_STAGE_BYTES;
            r_buf = r_buf == 2 ? 0 : r_buf + 1;
            r_sc += 4;
            ++r_s;
            if (r_s == r_nk || (r_s & 3) == 0) {                 // it starts a scale block (once per <= 4 steps)
                if (r_s == r_nk) {                               // ... of the next tile
                    r_tile += stride;
                    r_s = 0;
                    r_nk = r_tile < range_end ? tile_steps(r_tile) : 0x7FFFFFFF;
                }
                r_slot = r_slot == 2 ? 0 : r_slot + 1;
                // the last block of a K range is shifted back to end where the range ends
                const int within = r_s + 4 > r_nk ? r_s - (r_nk - 4) : 0;
                r_sc = Q_SCALE_OFF + r_slot * Q_SCALE_SLOT + within * 4;
            }
        }
        issue_and_wait();
        // (the compiler waits for the LDS reads here)
        const auto pa = __builtin_amdgcn_permlane32_swap(va, va, false, false);
        const auto pb0 = __builtin_amdgcn_permlane32_swap(vb0, vb0, false, false);
        const auto pb1 = __builtin_amdgcn_permlane32_swap(vb1, vb1, false, false);
        sca[0] = pa[0] >> 8 * lhalf; sca[1] = pa[1] >> 8 * lhalf;
        scb[0] = pb0[0] >> 8 * lhalf; scb[1] = pb0[1] >> 8 * lhalf;
        scb[2] = pb1[0] >> 8 * lhalf; scb[3] = pb1[1] >> 8 * lhalf;
        MX_PROBE(3);
    };
    // FIRST: the first K step of a tile; its first 64-K slice starts the accumulators from zero (the
    // matrix instruction takes a constant 0 as its addend), so they are never cleared by separate moves.
    auto mma_phase = [&](auto first_c) {
        constexpr bool FIRST = decltype(first_c)::value;
        MX_PROBE(4);
        MX_SCHED_FENCE();
        const v16f zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                v8i xa = v8i{f[kk].a[i].x, f[kk].a[i].y, f[kk].a[i].z, f[kk].a[i].w, 0, 0, 0, 0};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    v8i xb = v8i{f[kk].b[j].x, f[kk].b[j].y, f[kk].b[j].z, f[kk].b[j].w, 0, 0, 0, 0};
                    if (kk == 0)
                        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(xb, xa, FIRST ? zero : acc[i][j], 4, 4, 0, (int)scb[j], 0, (int)sca[i]);
                    else
                        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(xb, xa, acc[i][j], 4, 4, 2, (int)scb[j], 2, (int)sca[i]);
                }
            }
        MX_SCHED_FENCE();
        MX_PROBE(5);
    };
    // ---- prologue: stages 0 and 1 (scale block 0 travels with stage 0) ----
    set_issue_tile(first);
    issue_and_wait();
    issue_and_wait();                                                 // (ends with vmcnt(4): all but stage 1)
    asm volatile("s_barrier" ::: "memory");                           // stage 0 and scale block 0 are in
    if (GRP == 0) load_phase();                                       // operands of step 0

    // ---- per K step one barrier: group 0 runs  M(k) | barrier | L(k+1),  group 1 runs
    //      L(k) | barrier | M(k).  At the barrier every read of stage k has returned (group 0's were
    //      consumed by M(k), group 1 waits for its own), so the loads issued after it may overwrite
    //      that buffer; and every wave has waited for its part of stage k+1, which group 0 reads
    //      right after it.  Between barriers the two waves of a SIMD drift freely: one is in its
    //      MFMA burst while the other reads and loads. ----
    uint32_t c_bias = Q_BIAS_OFF;                                 // bias slot of the tile being multiplied
    for (uint32_t c_tile = first; c_tile < range_end; c_tile += stride) {
        const int nk = tile_steps(c_tile);
        // step 0 starts the accumulators, the others add to them (nk >= 4)
        if (GRP == 0) {
            mma_phase(std::true_type{});
            barrier_after_mfma(acc);
            load_phase();
        } else {
            load_phase();
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            mma_phase(std::true_type{});
        }
        for (int k = 1; k < nk; ++k) {
            if (GRP == 0) {
                mma_phase(std::false_type{});
                barrier_after_mfma(acc);
                load_phase();
            } else {
                load_phase();
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                mma_phase(std::false_type{});
            }
        }
        const uint32_t z = c_tile / tiles, r = c_tile - z * tiles, tm = r / g.tiles_n;
        const uint32_t m0 = tm * Q_BM + wm * 64, n0 = (r - tm * g.tiles_n) * Q_BN + GRP * 128;
        uint8_t* ep = (uint8_t*)(lds + Q_EP_OFF + wave * P_EP_BYTES);
        const lds_u8* bias = BIAS ? lds + c_bias + GRP * 512 : nullptr;
        const uint32_t c_bias_now = c_bias;
        if (BIAS) c_bias = c_bias == (uint32_t)Q_BIAS_OFF ? c_bias + 1024u : c_bias - 1024u;
        MX_PROBE(6);
        // wave tile wholly inside the matrix, rows storable 16 bytes at a time, lane offsets within 32 bits
        const bool final_out = g.split_k == 1;
        const int64_t ldc = final_out ? g.ldc : (int64_t)g.n;
        const uint32_t ebytes = (final_out && g.c_bf16) ? 2u : 4u;
        const bool interior = m0 + 64 <= g.m && n0 + 128 <= g.n && ldc < (1 << 27) &&
                              ((reinterpret_cast<uintptr_t>(g.c) | (uintptr_t)(ldc * ebytes)) & 15) == 0;
        if (interior) {
            if (final_out) gemm_epilogue_interior<true, BIAS>(g, lds + Q_EP_OFF + wave * P_EP_BYTES, acc, m0, n0, z, ldc, BIAS ? lds + c_bias_now + GRP * 512 : nullptr);
            else           gemm_epilogue_interior<false, false>(g, lds + Q_EP_OFF + wave * P_EP_BYTES, acc, m0, n0, z, ldc, nullptr);
        } else {
            if (final_out) gemm_epilogue_chunked<true>(g, ep, acc, m0, n0, lane, z, bias);
            else           gemm_epilogue_chunked<false>(g, ep, acc, m0, n0, lane, z, nullptr);
        }
        if (GELUQ) {
            // BIAS is set with GELUQ: the bias slot of this tile is still valid (it is reused two tiles later)
            if (g.q_floor) gemm_epilogue_gelu_quant<true>(g, lds + Q_EP_OFF + wave * P_EP_BYTES, acc, m0, n0, lds + c_bias_now + GRP * 512);
            else           gemm_epilogue_gelu_quant<false>(g, lds + Q_EP_OFF + wave * P_EP_BYTES, acc, m0, n0, lds + c_bias_now + GRP * 512);
        }
        MX_PROBE(7);
    }
    // the cursor's trailing loads target this workgroup's LDS: they must land before it is released
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// BIAS: a bias row is added in the output stage (a separate instance: the plain product's code is
// the same with and without this feature in the source).
// GELUQ (only with BIAS): a second output stage quantizes GELU(product + bias) for the next layer.
template <bool BIAS, bool GELUQ = false>
__global__ __launch_bounds__(Q_NT, 2) void mx_gemm_pingpong_kernel(GemmArgs g)
{
    __shared__ __attribute__((aligned(1024))) uint8_t lds[BIAS ? Q_LDS_BYTES : Q_BIAS_OFF];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Short-K tiles spend as long storing as multiplying.  Started together, all compute units store
    // at the same time, the burst (33 MB per round) takes longer to drain than the next K loop has
    // loads in flight for, and the loop stalls behind it; the stalled units then stay in step.  Half
    // of the workgroups start half a K loop later, so that one half stores while the other multiplies.
    if ((blockIdx.x >> 3) & 1)
        for (int i = 0; i < g.stagger; ++i) __builtin_amdgcn_s_sleep(32);
    if (wave < 4) pingpong_wave<0, BIAS, GELUQ>(g, (lds_u8*)lds, wave);
    else          pingpong_wave<1, BIAS, GELUQ>(g, (lds_u8*)lds, wave);
}

// ---------------------------------------------------------------------------
// Calibration: the products' MFMA in a register-resident loop.  8 waves per workgroup (two per
// SIMD, as in the main kernel), each with the main kernel's 8 independent accumulator tiles; every lane
// loads its 12 operand registers (two 64-K slices of 2 m-side and 4 n-side fragments) once from the
// caller's buffer and then issues 16 MFMAs per iteration with no memory or LDS access in between.
// What it measures is the rate the matrix pipe sustains for these operand bytes; that rate depends
// on the bytes (switching activity against the power limit), which is why the caller supplies them.
// ---------------------------------------------------------------------------
constexpr int CAL_WAVES = 8, CAL_FRAGS = 12;
constexpr size_t CAL_OPERAND_BYTES = (size_t)CAL_WAVES * CAL_FRAGS * 64 * 16;      // 98304

__global__ __launch_bounds__(CAL_WAVES * 64, 1) void calibration_mfma_kernel(const v4i* __restrict__ operands, int iterations,
                                                                            float* sink)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    v4i f[CAL_FRAGS];
#pragma unroll
    for (int q = 0; q < CAL_FRAGS; ++q) f[q] = operands[(wave * CAL_FRAGS + q) * 64 + lane];
    v16f acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    for (int it = 0; it < iterations; ++it) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const v4i a = f[kk * 6 + i];
                const v8i xa = v8i{a.x, a.y, a.z, a.w, 0, 0, 0, 0};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const v4i b = f[kk * 6 + 2 + j];
                    const v8i xb = v8i{b.x, b.y, b.z, b.w, 0, 0, 0, 0};
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(xb, xa, acc[i][j], 4, 4, 0, 0x7F7F7F7F, 0, 0x7F7F7F7F);
                }
            }
        MX_SCHED_FENCE();
    }
    // keep the accumulators alive; one value per lane leaves the kernel
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) t += acc[i][j][r];
    sink[(size_t)blockIdx.x * (CAL_WAVES * 64) + threadIdx.x] = t;
}

}  // namespace

namespace mxl {

size_t calibration_mfma_operand_bytes() { return CAL_OPERAND_BYTES; }

hipError_t launch_calibration_mfma(const uint8_t* operands, int workgroups, int iterations, float* sink, hipStream_t st)
{
    hipLaunchKernelGGL(calibration_mfma_kernel, dim3((unsigned)workgroups), dim3(CAL_WAVES * 64), 0, st,
                       reinterpret_cast<const v4i*>(operands), iterations, sink);
    return hipGetLastError();
}

// Which kernel a product runs on and how many K splits it has.  The lines between the kernels come from a
// sweep of m = 64..25216, n = 192..3072, K = 192..50432 on the card (us, each product alone in a replayed graph):
//   main kernel: enough 256 x 256 tiles to occupy half the compute units (12672 x 768 x 768: 10.6 against 11.8 on
//     128 x 128 tiles, 25216 x 1536 x 3072: 79 against 131), or enough work for a K split of them
//     (768 x 768 x 50432: 36 against 42 and 46; at 1.5e10 multiply-adds it is even, 768 x 768 x 25216: 29 and 29).
//     Not where K is short and its second round would be less than a quarter full (25216 x 768 x 512: 16.4 against 15.3 on
//     128 x 128 tiles, 9856 x 2048 x 512 16.5 / 14.7, 6304 x 3072 x 768 19.7 / 19.0; 25216 x 768 x 1024 22.6 / 22.5).
//   64 x 64 tiles: up to one tile per compute unit (224 x 192 x 768: 4.1 against 6.6 on 128 x 128 and 8.0 on the
//     main kernel), with a K split up to two per unit (768 x 192 x 12672: 11 against 13 and 18).
//   128 x 64 tiles: up to three per unit (9856 x 384 x 1536: 9.4 against 11.3 and 12.3).
//   128 x 128 tiles: what is left, i.e. long m or n at K < 512 or K % 128 != 0; with all of K in one step for 256 < K <=
//     384 (bf16 25216 x 1536 x 384 22.4 against 24.5, FP32 25216 x 1152 x 384 27.5 against 30.0, 12608 x 1024 x 352 15.7
//     against 17.1), where steps of 128 wait three times; up to 256 it only takes LDS (12608 x 576 x 192 6.8 against 6.65).
// K splits (K >= 4096): s partials cost s * m * n * 4 bytes written and read, the K loop is K / s long; the sum is
// least at s ~ sqrt(K / (m n)) times the constant below, measured per kernel, within the slots of one round.
enum class GemmKernel { pingpong, tile128, tile128_short, tile128x64, tile64 };

struct GemmPlan {
    GemmKernel kernel;
    int split_k;
};

static GemmPlan plan_gemm(int64_t m, int64_t n, int64_t k)
{
    auto tiles = [&](int64_t bm, int64_t bn) -> int64_t { return ((m + bm - 1) / bm) * ((n + bn - 1) / bn); };
    const double mn = (double)m * (double)n, ratio = std::sqrt((double)k / mn);
    auto splits = [&](int64_t slots, int64_t count, double scale, int64_t min_k) -> int {
        if (k < 4096) return 1;
        const int64_t s = std::min({slots / count, k / min_k, (int64_t)(scale * ratio), (int64_t)64});
        return s < 1 ? 1 : (int)s;
    };
    const int64_t t256 = tiles(Q_BM, Q_BN), t12864 = tiles(128, 64), t64 = tiles(64, 64);
    const bool main_ok = (k & 127) == 0 && k >= 512;
    if (main_ok && k <= 768 && t256 > (int64_t)Q_SLOTS && t256 * 100 < 2 * (int64_t)Q_SLOTS * 62) return {GemmKernel::tile128, 1};
    if (main_ok && (t256 >= 128 || mn * (double)k >= 1.6e10))
        return {GemmKernel::pingpong, t256 * 2 <= 256 ? splits(256, t256, 60.0, 1024) : 1};
    if (t64 <= (k >= 4096 ? 512 : 256)) return {GemmKernel::tile64, splits(512, t64, 24.0, 1024)};
    if (t12864 <= 768) return {GemmKernel::tile128x64, splits(768, t12864, 35.0, 1024)};
    if (main_ok) return {GemmKernel::pingpong, 1};
    return {k > 256 && k <= 384 ? GemmKernel::tile128_short : GemmKernel::tile128, 1};
}

int gemm_split_k(int64_t m, int64_t n, int64_t k) { return plan_gemm(m, n, k).split_k; }

bool gemm_takes_fused_quantizer(int64_t m, int64_t n, int64_t k)
{
    // K a multiple of 128 with at least four K steps (what the main kernel takes), without a K split: a long K
    // with fewer than half the units' worth of 256 x 256 tiles is a K-split product's shape.
    return (k & 127) == 0 && k >= 512 && (n & 31) == 0 &&
           (k < 4096 || ((m + Q_BM - 1) / Q_BM) * ((n + Q_BN - 1) / Q_BN) * 2 > 256);
}

// Kernel of a product with the fused GELU stage (no K split).  All give the same bytes.  The main kernel takes 25 us for
// any number of tiles up to one per compute unit, because both wave groups of a unit go through the stage at once; with
// 64 x 64 tiles up to two rounds of 512 take 9-13 us, with 128 x 128 tiles waves of three workgroups share a unit and one
// multiplies while another is in the stage.  Main kernel / 128 x 128 / 64 x 64 tiles in us (m x n x k):
//   224x3072x768 24 13 9    1312x3072x1024 26 19 15    2048x3072x1024 26 19.9 20.4    6304x3072x1024 53 38 -
//   25216x2048x640 93 75    25216x3072x768 120 110     50432x3072x768 229 220         25216x1280x896 57 56
//   40000x1024x896 76 63    25216x3072x1024 126 129    8000x1536x1024 28.6 27.5       25216x3072x2048 162 196
//   6304x3072x2048 64 57    3136x3072x3072 39 49
// and where one round of the main kernel holds all tiles and is well filled (medians of 13 such sizes: 1.00 at K = 512, 1.02
// at 640, 1.04 at 768, 1.06 at 896):
//   12608x1024x512 25.5 25.1    8192x2048x512 27.1 27.5    4096x4096x640 29.1 29.1    8192x2048x640 28.5 29.3
//   12608x1024x768 27.1 28.1    6400x2560x768 29.6 31.3    16384x1024x896 30.7 32.7   5120x3072x896 29.9 32.1
// 128 x 128 tiles win where the main kernel's rounds of 256 tiles would be filled to less than 70 % and K is not long, and
// up to K = 896 wherever there is more than one round; with one, it is even up to K = 640 and the main kernel wins beyond.
static GemmKernel plan_fused(int64_t m, int64_t n, int64_t k)
{
    if (((m + 63) / 64) * ((n + 63) / 64) <= 1024) return GemmKernel::tile64;
    const int64_t t256 = ((m + Q_BM - 1) / Q_BM) * ((n + Q_BN - 1) / Q_BN), rounds = (t256 + Q_SLOTS - 1) / Q_SLOTS;
    if (k <= 2048 && t256 * 10 < rounds * Q_SLOTS * 7) return GemmKernel::tile128;
    return k <= (rounds > 1 ? 896 : 640) ? GemmKernel::tile128 : GemmKernel::pingpong;
}

const char* gemm_kernel_name(int64_t m, int64_t n, int64_t k, bool fused)
{
    if (fused && !gemm_takes_fused_quantizer(m, n, k)) return "none";
    switch (fused ? plan_fused(m, n, k) : plan_gemm(m, n, k).kernel) {
    case GemmKernel::pingpong: return "main";
    case GemmKernel::tile128: return "128x128";
    case GemmKernel::tile128_short: return "128x128 in one step";
    case GemmKernel::tile128x64: return "128x64";
    case GemmKernel::tile64: return "64x64";
    }
    return "none";
}

// Kernel arguments of a product and the kernel that it runs on; the tile counts are filled in by tile_grid().
static GemmKernel make_gemm_args(const GemmParams& p, GemmArgs& g)
{
    g = GemmArgs{};
    g.a_codes = p.a_codes; g.a_scales = p.a_scales; g.b_codes = p.b_codes; g.b_scales = p.b_scales;
    g.m = (uint32_t)p.m; g.n = (uint32_t)p.n; g.k = (uint32_t)p.k;
    const uint32_t ksteps = (uint32_t)((p.k + 127) / 128);
    const uint32_t steps_per = (ksteps + p.split_k - 1) / p.split_k;
    g.k_per_split = steps_per * 128;
    g.split_k = (int)((ksteps + steps_per - 1) / steps_per);   // drop empty splits
    g.c = g.split_k > 1 ? p.workspace : p.c;
    g.ldc = p.ldc; g.c_bf16 = p.c_bf16;
    g.bias = g.split_k > 1 ? nullptr : p.bias;                  // partial sums get none: the reduction adds it
    GemmKernel kernel = p.q_codes ? plan_fused(p.m, p.n, p.k) : plan_gemm(p.m, p.n, p.k).kernel;
    // the main kernel needs four K steps in every split (the last one may be short of that)
    if (kernel == GemmKernel::pingpong && ksteps - (uint32_t)(g.split_k - 1) * steps_per < 4) kernel = GemmKernel::tile128;
    return kernel;
}

static unsigned tile_grid(GemmArgs& g, uint32_t bm, uint32_t bn)
{
    g.tiles_m = (g.m + bm - 1) / bm;
    g.tiles_n = (g.n + bn - 1) / bn;
    return g.tiles_m * g.tiles_n * (unsigned)g.split_k;
}

// Start delay of every other workgroup of the main kernel.  Measured on the ViT-B products: 2.5 us (3 x 2048 clocks) gains
// 5-15 % at K = 768 and 3-5 % at K = 2304, nothing at K = 3072; pointless below two rounds of tiles.
static int stagger_of(const GemmArgs& g, unsigned tiles) { return (g.split_k == 1 && tiles >= 2 * Q_SLOTS && g.k <= 2304) ? 3 : 0; }

// What is left of a product after its kernel: the sum over a K split, and the column sums.
static hipError_t finish_product(const GemmParams& p, const GemmArgs& g, hipStream_t st, const ColumnSumTail* tail)
{
    if (g.split_k > 1) {
        size_t total = (size_t)p.m * p.n;
        const size_t out_bytes = p.c_bf16 ? 2 : 4;
        const bool vec = (p.n & 3) == 0 && ((size_t)p.ldc * out_bytes & 15) == 0 &&
                         (reinterpret_cast<uintptr_t>(p.c) & 15) == 0 && (reinterpret_cast<uintptr_t>(p.workspace) & 15) == 0;
        const unsigned blocks = (unsigned)(((vec ? total / 4 : total) + 255) / 256);
        const ColumnSumTail t = tail ? *tail : ColumnSumTail{};
        const unsigned tail_blocks = (t.cols + 31) / 32;
        const dim3 rgrid(blocks + tail_blocks), rblock(256);
        if (vec)
            hipLaunchKernelGGL(splitk_reduce4_kernel, rgrid, rblock, 0, st, static_cast<const float*>(p.workspace), g.split_k, g.m, g.n,
                               p.c, p.ldc, (int)p.c_bf16, p.bias, t, tail_blocks);
        else
            hipLaunchKernelGGL(splitk_reduce_kernel, rgrid, rblock, 0, st, static_cast<const float*>(p.workspace), g.split_k, g.m, g.n,
                               p.c, p.ldc, (int)p.c_bf16, p.bias, t, tail_blocks);
        return hipGetLastError();
    }
    return tail && tail->cols ? launch_column_sum_finish(*tail, st) : hipSuccess;
}

hipError_t launch_gemm(const GemmParams& p, hipStream_t st, const ColumnSumTail* tail)
{
    GemmArgs g;
    const GemmKernel kernel = make_gemm_args(p, g);
    if (p.q_codes) {
        if (!gemm_takes_fused_quantizer(p.m, p.n, p.k) || !g.bias || g.split_k != 1) return hipErrorInvalidValue;
        g.q_codes = p.q_codes; g.q_scales = p.q_scales; g.q_floor = p.q_floor ? 1 : 0;
    }
    switch (kernel) {
    case GemmKernel::pingpong: {
        const unsigned nblk = tile_grid(g, Q_BM, Q_BN);
        g.stagger = stagger_of(g, nblk);
        const dim3 pgrid(nblk < Q_SLOTS ? nblk : Q_SLOTS);
        if (p.q_codes) {
            hipLaunchKernelGGL((mx_gemm_pingpong_kernel<true, true>), pgrid, dim3(Q_NT), 0, st, g);
        } else if (g.bias) {
            hipLaunchKernelGGL(mx_gemm_pingpong_kernel<true>, pgrid, dim3(Q_NT), 0, st, g);
        } else {
            hipLaunchKernelGGL(mx_gemm_pingpong_kernel<false>, pgrid, dim3(Q_NT), 0, st, g);
        }
        break;
    }
    case GemmKernel::tile128:
        if (p.q_codes) hipLaunchKernelGGL((mx_gemm_tile_kernel<Tile128, true>), dim3(tile_grid(g, 128, 128)), dim3(T_NT), 0, st, g);
        else           hipLaunchKernelGGL(mx_gemm_tile_kernel<Tile128>, dim3(tile_grid(g, 128, 128)), dim3(T_NT), 0, st, g);
        break;
    case GemmKernel::tile128_short:
        hipLaunchKernelGGL(mx_gemm_tile_kernel<Tile128Short>, dim3(tile_grid(g, 128, 128)), dim3(T_NT), 0, st, g);
        break;
    case GemmKernel::tile128x64:
        hipLaunchKernelGGL(mx_gemm_tile_kernel<Tile128x64>, dim3(tile_grid(g, 128, 64)), dim3(T_NT), 0, st, g);
        break;
    case GemmKernel::tile64:
        if (p.q_codes) hipLaunchKernelGGL((mx_gemm_tile_kernel<Tile64, true>), dim3(tile_grid(g, 64, 64)), dim3(T_NT), 0, st, g);
        else           hipLaunchKernelGGL(mx_gemm_tile_kernel<Tile64>, dim3(tile_grid(g, 64, 64)), dim3(T_NT), 0, st, g);
        break;
    }
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? finish_product(p, g, st, tail) : e;
}

// One tile per compute unit and two K steps at most.  Device time of one MxLinear call without gradients, separate kernels /
// this one, in a replayed graph, in us (m x k -> n, X / W):
//   197 x 192 -> 768    bf16 / FP32 6.3 / 5.1    1000 x 256 -> 1024  FP32 / FP32 6.6 / 5.9    32 x 32 -> 64  bf16 / bf16 5.2 / 4.5
//   512 x 384 -> 384    bf16 / FP32 6.0 / 7.1    2000 x 512 -> 512   bf16 / FP32 6.5 / 7.7    1 x 288 -> 1024 FP32 / FP32 6.3 / 7.3
//   8192 x 512 -> 64    FP32 / FP32 8.4 / 7.7    16384 x 384 -> 64   bf16 / FP32 8.3 / 7.6    64 x 512 -> 4096 bf16 / bf16 7.4 / 6.9
// Up to 256 columns it is faster at every size and type (0.67 to 0.94 of the separate kernels' time).  A second K step costs
// 1.8 us (a unit quantizes 128 x 256 values for it) and loses that, except where the separate quantizer takes long: an X of
// about 3.5 M elements and more, and a bf16 bias of 3072 values and more, which one workgroup of that launch widens.
// A call by itself is bound by the host (512 x 384 -> 384: 10.0 us with two launches, 6.8 with one), which a recorded graph
// leaves behind: only a call that is being captured goes by the device time.
bool linear_fits_one_launch(int64_t m, int64_t n, int64_t k, bool bias_bf16, bool captured)
{
    if (((m + 63) / 64) * ((n + 63) / 64) > 256 || k > 512) return false;
    return k <= 256 || !captured || m * k >= (7 << 19) || (bias_bf16 && n >= 3072);
}

hipError_t launch_quantized_linear(const QuantizedLinearParams& p, hipStream_t st)
{
    QuantizedLinearArgs a{};
    a.x = p.x; a.w = p.w; a.bias = p.bias; a.bias_bf16 = p.bias_bf16;
    a.g.m = (uint32_t)p.m; a.g.n = (uint32_t)p.n; a.g.k = (uint32_t)p.k;
    a.g.split_k = 1; a.g.k_per_split = a.g.k;
    a.g.c = p.c; a.g.c_bf16 = p.c_bf16; a.g.ldc = p.n;
    const dim3 grid(tile_grid(a.g, 64, 64)), block(QL_NT);
    auto launch = [&](auto x, auto w) {
        using XT = decltype(x);
        using WT = decltype(w);
        if (p.floor_mode) hipLaunchKernelGGL((mx_quantized_linear_kernel<XT, WT, true>), grid, block, 0, st, a);
        else              hipLaunchKernelGGL((mx_quantized_linear_kernel<XT, WT, false>), grid, block, 0, st, a);
    };
    if (p.x_bf16) {
        if (p.w_bf16) launch(uint16_t{}, uint16_t{});
        else          launch(uint16_t{}, float{});
    } else {
        if (p.w_bf16) launch(float{}, uint16_t{});
        else          launch(float{}, float{});
    }
    return hipGetLastError();
}

// Two independent products of a backward pass, w and x, in one launch where both run on tile kernels and have a workspace
// each (or need one at most): alone each fills its last round sparsely, or the chip altogether, and waits for the one
// before.  Never slower at 120 pairs timed (32 to 25216 tokens, 128 to 1536 columns, 128 to 4000 outputs, FP32 and bf16: 0.73
// to 1.00 of the time apart), though both then have the LDS of the larger shape; quantizer, both products and
// reduction of MxLinearStep.backward in a replayed graph, apart / together in us: 256 x 192 -> 768 FP32 13.0 / 9.9,
// 1024 x 768 -> 3072 25.5 / 20.4, 6304 x 192 -> 576 24.6 / 20.9, 25216 x 384 -> 384 42.5 / 36.9, 12608 x 192 -> 768
// 38.8 / 36.4, 25216 x 1536 -> 384 80.7 / 74.7, bf16 3744 x 1504 -> 2208 55.8 / 54.4, 15520 x 1344 -> 672 68.8 / 68.2.
// Where the main kernel takes one of them they stay apart: a tile kernel in its place costs what is gained
// (12608 x 768 -> 2304 82 / 90, 6304 x 1024 -> 1024 42 / 37), and two products on the main kernel leave each other
// nothing (50432 x 2304 x 768 with 768 x 2304 x 50432: 116 apart, 124 together: its units are handed over one by one).
// (w on 128 x 128 tiles: a large weight and few tokens, which fill the chip by themselves)
static bool pair_on_tile_kernels(GemmKernel kw, GemmKernel kx)
{
    return (kw == GemmKernel::tile64 || kw == GemmKernel::tile128x64) && kx != GemmKernel::pingpong;
}

bool gemm_pair_fits_one_launch(const GemmParams& w, const GemmParams& x)
{
    GemmArgs g;
    return !w.q_codes && !x.q_codes && pair_on_tile_kernels(make_gemm_args(w, g), make_gemm_args(x, g));
}

hipError_t launch_gemm_pair(const GemmParams& w, const GemmParams& x, hipStream_t st, const ColumnSumTail* tail)
{
    GemmArgs gw, gx;
    const GemmKernel kw = make_gemm_args(w, gw), kx = make_gemm_args(x, gx);
    // two K splits with one workspace: the partial sums of one must have been added up before the other writes its own
    const bool own_scratch = gw.split_k == 1 || gx.split_k == 1 || w.workspace != x.workspace;
    if (!own_scratch || !pair_on_tile_kernels(kw, kx) || w.q_codes || x.q_codes) {
        const hipError_t e = launch_gemm(x, st);
        return e == hipSuccess ? launch_gemm(w, st, tail) : e;
    }
    auto launch = [&](auto sw, auto sx) {
        using SW = decltype(sw);
        using SX = decltype(sx);
        const unsigned nw = tile_grid(gw, SW::BM, SW::BN), nx = tile_grid(gx, SX::BM, SX::BN), first = (nw + 7u) / 8u * 8u;
        hipLaunchKernelGGL((mx_gemm_tile_pair_kernel<SW, SX>), dim3(first + nx), dim3(T_NT), 0, st, gw, gx, first);
    };
    auto with_x = [&](auto sw) {
        if (kx == GemmKernel::tile64)          launch(sw, Tile64{});
        else if (kx == GemmKernel::tile128x64) launch(sw, Tile128x64{});
        else if (kx == GemmKernel::tile128)    launch(sw, Tile128{});
        else                                   launch(sw, Tile128Short{});
    };
    if (kw == GemmKernel::tile64) with_x(Tile64{});
    else                          with_x(Tile128x64{});
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = finish_product(x, gx, st, nullptr);
    return e == hipSuccess ? finish_product(w, gw, st, tail) : e;
}

}  // namespace mxl
