// Q-Ramping's customised AdamW (Algorithm 2; Sec. 6.2) for gfx950: one streaming pass over the
// weights of the quantized layers, bound by memory.
//
// A weight element with amplification factor N_w has N_w times the global batch size -- its
// gradient is accumulated over N_w steps -- and N_w times the global learning rate.  Per element
// and step:
//     g_acc += grad;  acc_steps += 1;
//     if acc_steps >= N_w:
//         g = g_acc / acc_steps;  lr_w = N_w * lr;  u = ++updates;
//         w = w * (1 - lr_w * weight_decay)
//         m = beta1 * m + (1 - beta1) * g;   v = beta2 * v + (1 - beta2) * g * g
//         w = w - (lr_w / (1 - beta1^u)) * m / (sqrt(v) / sqrt(1 - beta2^u) + eps)
//         g_acc = 0;  acc_steps = 0
// An element with factor N thus follows AdamW at learning rate N * lr on the means of N consecutive
// gradients, with the bias correction counting its own updates.  FP32 arithmetic; 1 - beta and
// ln(beta) come from the host in double precision, and 1 - beta^u = -expm1(u * ln(beta)) keeps its
// relative accuracy when u is small.
//
// Work split: one launch serves up to 32 (in a detection window 24) tensors, whose addresses travel in the kernel's
// arguments; a ViT's step is then 2 to 5 launches instead of one to four per parameter (ViT-Tiny, 144 parameters:
// 240 launches of 3-5 us each for 5.3 M elements).  A lane owns 4 consecutive elements (16-byte accesses on every
// array), in a detection window two times 4; eight lanes there hold a 1x32 group.
//
// Bytes per element: 28 read + 16 written where no gradient is held.  The held sum is read only by lanes whose step
// count is not zero (the two are zero together, an element's update clears both), and sum and count are written only
// where they change, so the weights with factor 1 -- all but a few percent -- cost 44 B instead of 56.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cmath>
#include <cstdint>
#include "mx_device.hpp"
#include "mx_launch.hpp"

namespace {

constexpr int OPT_THREADS = 256;

typedef float v4f __attribute__((ext_vector_type(4)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));

struct AdamHyper {
    float lr, beta1, beta2, eps, weight_decay;
    float one_minus_beta1, one_minus_beta2, ln_beta1, ln_beta2;
};

AdamHyper hyper_of(float lr, float beta1, float beta2, float eps, float weight_decay)
{
    AdamHyper h{};
    h.lr = lr; h.beta1 = beta1; h.beta2 = beta2; h.eps = eps; h.weight_decay = weight_decay;
    h.one_minus_beta1 = (float)(1.0 - (double)beta1);
    h.one_minus_beta2 = (float)(1.0 - (double)beta2);
    h.ln_beta1 = (float)std::log((double)beta1);
    h.ln_beta2 = (float)std::log((double)beta2);
    return h;
}

// every array is touched once per step and the state of a model is far larger than the
// last-level cache: all accesses are marked streaming
__device__ __forceinline__ v4f load4(const float* p, int64_t q) { return __builtin_nontemporal_load(reinterpret_cast<const v4f*>(p) + q); }
__device__ __forceinline__ v4i load4(const int32_t* p, int64_t q) { return __builtin_nontemporal_load(reinterpret_cast<const v4i*>(p) + q); }
__device__ __forceinline__ void store4(float* p, int64_t q, v4f v) { __builtin_nontemporal_store(v, reinterpret_cast<v4f*>(p) + q); }
__device__ __forceinline__ void store4(int32_t* p, int64_t q, v4i v) { __builtin_nontemporal_store(v, reinterpret_cast<v4i*>(p) + q); }

__device__ __forceinline__ v4f load_grad4(const void* g, bool bf16, int64_t q)
{
    if (!bf16) return load4(static_cast<const float*>(g), q);
    const v2u r = __builtin_nontemporal_load(static_cast<const v2u*>(g) + q);
    return v4f{__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xFFFF0000u), __uint_as_float(r.y << 16), __uint_as_float(r.y & 0xFFFF0000u)};
}

// What an update needs besides the gradient, for an element that makes its u-th update with factor n_w.
struct StepScale { float lr_w, step_size, root_bc2; };

__device__ __forceinline__ StepScale step_scale(const AdamHyper& a, int32_t u, int32_t n_w)
{
    const float bc1 = -expm1f((float)u * a.ln_beta1);
    const float bc2 = -expm1f((float)u * a.ln_beta2);
    const float lr_w = (float)n_w * a.lr;
    return {lr_w, __fdiv_rn(lr_w, bc1), __fsqrt_rn(bc2)};
}

__device__ __forceinline__ void adamw_update(const AdamHyper& a, float& w, float& m, float& v, float gm, const StepScale& k)
{
    w = w * (1.0f - k.lr_w * a.weight_decay);
    m = a.beta1 * m + a.one_minus_beta1 * gm;
    v = a.beta2 * v + a.one_minus_beta2 * gm * gm;
    const float denom = __fdiv_rn(__fsqrt_rn(v), k.root_bc2) + a.eps;
    w = w - __fdiv_rn(k.step_size * m, denom);
}

// Whether the four elements of every lane of the wave have made the same number of updates and take this one at
// factor 1 with nothing held (then u is that number).  The bias corrections -- two expm1, a square root, a division --
// are then computed once per lane instead of once per element.
__device__ __forceinline__ bool uniform_updates(const v4i& u)
{
    const int first = __builtin_amdgcn_readfirstlane(u.x);
    return __all(u.x == first && u.y == first && u.z == first && u.w == first);
}

// Whether p holds in any of the eight lanes whose quads share a 128-byte line.  Stores are decided by line: a line of which
// some lanes write nothing is a partial write, which the memory turns into a read and a write (factors 1 to 6 at random on
// 84 M elements: 1042 us with stores decided by lane, 839 when every array was written).
__device__ __forceinline__ bool any_of_line(bool p)
{
    const uint64_t b = __builtin_amdgcn_ballot_w64(p);
    return ((b >> (threadIdx.x & 56u)) & 0xFFu) != 0u;
}

constexpr int ADAM_BATCH = mxl::ADAM_BATCH_MAX;

struct AdamTensor {
    float* w;
    const void* grad;
    float* m;
    float* v;
    int32_t* updates;
    float* g_acc;                 // null iff factor is null
    const int32_t* factor;        // null: 1 everywhere
    int32_t* acc_steps;           // null iff factor is null
};

// N: 1 or ADAM_BATCH.  The arguments of 32 tensors are 2.4 KB, which cost a launch of one tensor a microsecond.
template <int N>
struct AdamBatch {
    AdamHyper h;
    uint32_t grad_bf16;           // bit i: tensor i's gradient
    uint32_t end[N];              // first workgroup past tensor i
    int64_t quads[N];             // count / 4
    AdamTensor t[N];
};

template <bool RAMPING, int N>
__global__ __launch_bounds__(OPT_THREADS) void ramping_adamw_kernel(AdamBatch<N> b)
{
    uint32_t i = 0;
#pragma unroll
    for (int k = 0; k + 1 < N; ++k) i += blockIdx.x >= b.end[k] ? 1u : 0u;
    const AdamTensor t = b.t[i];
    const AdamHyper& a = b.h;
    const int64_t q = (int64_t)(blockIdx.x - (i ? b.end[i - 1] : 0u)) * OPT_THREADS + threadIdx.x;
    if (q >= b.quads[i]) return;
    v4f w = load4(t.w, q), m = load4(t.m, q), v = load4(t.v, q);
    const v4f g = load_grad4(t.grad, (b.grad_bf16 >> i) & 1u, q);
    v4i u = load4(t.updates, q);
    if (RAMPING) {
        const v4i n = load4(t.factor, q);
        v4i c = load4(t.acc_steps, q);
        const bool plain = n.x == 1 && n.y == 1 && n.z == 1 && n.w == 1 && (c.x | c.y | c.z | c.w) == 0;
        if (!__all(plain) || !uniform_updates(u)) {
            v4f acc = {0.f, 0.f, 0.f, 0.f};
            const bool held = (c.x | c.y | c.z | c.w) != 0;
            if (held) acc = load4(t.g_acc, q);
            bool any = false;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[e] = acc[e] + g[e];
                c[e] += 1;
                if (c[e] < n[e]) continue;                  // this element's batch is not full yet
                any = true;
                u[e] += 1;
                float we = w[e], me = m[e], ve = v[e];
                adamw_update(a, we, me, ve, __fdiv_rn(acc[e], (float)c[e]), step_scale(a, u[e], n[e]));
                w[e] = we; m[e] = me; v[e] = ve;
                acc[e] = 0.0f;
                c[e] = 0;
            }
            if (any_of_line(any)) {
                store4(t.w, q, w);
                store4(t.m, q, m);
                store4(t.v, q, v);
                store4(t.updates, q, u);
            }
            if (any_of_line(held || (c.x | c.y | c.z | c.w) != 0)) {
                store4(t.g_acc, q, acc);
                store4(t.acc_steps, q, c);
            }
            return;
        }
    }
    // factor 1, nothing held
    if (uniform_updates(u)) {
        const StepScale k = step_scale(a, u.x + 1, 1);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float we = w[e], me = m[e], ve = v[e];
            adamw_update(a, we, me, ve, 0.0f + g[e], k);
            w[e] = we; m[e] = me; v[e] = ve;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float we = w[e], me = m[e], ve = v[e];
            adamw_update(a, we, me, ve, 0.0f + g[e], step_scale(a, u[e] + 1, 1));
            w[e] = we; m[e] = me; v[e] = ve;
        }
    }
    u += 1;
    store4(t.w, q, w);
    store4(t.m, q, m);
    store4(t.v, q, v);
    store4(t.updates, q, u);
}

// One step inside a detection window: the AdamW step at factor 1 (gradients still held are applied with it), the 1x32
// quantization of the new weight and the step of the trajectory lengths dist_W, dist_Q (Sec. 6.1), in one pass:
// w crosses memory once instead of four times and the codes are not read back.  The arithmetic is that of
// ramping_adamw_kernel, quantize_rows_kernel (round_D) and oscillation_kernel.  `opens` (the window's first step): the
// lengths start from the weight as it is before the step.
constexpr int WINDOW_BATCH = mxl::WINDOW_BATCH_MAX;

struct WindowBatch {
    AdamHyper h;
    uint32_t grad_bf16;
    int opens;
    uint32_t end[WINDOW_BATCH];
    uint32_t quads[WINDOW_BATCH];       // count / 4, a multiple of 8
    mxl::WindowTensor t[WINDOW_BATCH];
};

// round_D codes (16 bits) of a lane's 4 elements of a group of 8 lanes, and the group's scale byte
template <bool FLOOR>
__device__ __forceinline__ uint32_t rtn_codes4(const v4f& x, uint32_t& byte)
{
    using namespace mxd;
    uint32_t m = quad_max(absmax3_bits(x.x, x.y, absmax3_bits(x.z, x.w, 0u)));
    const uint32_t other = (uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0x141, 0xF, 0xF, true);      // row_half_mirror: the other four lanes
    m = m > other ? m : other;
    byte = scale_byte(m, FLOOR);
    const float s = scale_operand(byte);
    return cvt_rtn_f32<1>(cvt_rtn_f32<0>(x.x, x.y, s), x.z, x.w, s) & 0xFFFFu;
}

__device__ __forceinline__ v4f dequantize4(uint32_t codes, uint32_t byte)
{
    using namespace mxd;
    const float s = scale_operand(byte);
    const f32x2_hw a = cvt_f32_fp4<0>(codes, s), b = cvt_f32_fp4<1>(codes, s);
    return v4f{a.x, a.y, b.x, b.y};
}

// A lane owns two quads of 4 elements, 64 quads apart, so that every access of a wave is one run of 1 KB (64 bytes to 1 KB
// for the packed arrays).  With 8 neighbouring elements in a lane instead, each instruction takes every other 16 bytes, and
// streaming loads and stores do not meet in the cache: 2.65 M elements 52 us, 3.1 TB/s; as two quads 33.7 us, 5.1 TB/s.
constexpr int WINDOW_QUADS = 2;

template <bool FLOOR>
__global__ __launch_bounds__(OPT_THREADS) void ramping_window_kernel(WindowBatch b)
{
    uint32_t i = 0;
#pragma unroll
    for (int k = 0; k + 1 < WINDOW_BATCH; ++k) i += blockIdx.x >= b.end[k] ? 1u : 0u;
    const mxl::WindowTensor t = b.t[i];
    const AdamHyper& a = b.h;
    const uint32_t quads = b.quads[i];
    const uint32_t q0 = (blockIdx.x - (i ? b.end[i - 1] : 0u)) * (OPT_THREADS * WINDOW_QUADS) + (threadIdx.x & ~63u) * WINDOW_QUADS + (threadIdx.x & 63u);
    // every load before the first store: the arrays could overlap for all the compiler knows, and a wave that waits
    // for its stores before it loads again reaches half the memory rate.  Past the end the last quad is read again and
    // nothing is stored (quads % 8 == 0: the eight lanes of a group stay together).
    const bool has_grad = t.grad != nullptr;            // a weight without a gradient stands still
    constexpr int H = WINDOW_QUADS;
    v4f w[H], prev[H], dw[H], dq[H], g[H], m[H], v[H], acc[H];
    v4i u[H], c[H];
    uint32_t byte[H], codes_prev[H];
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const int64_t q = min(q0 + 64u * h, quads - 1u);
        w[h] = load4(t.w, q);
        if (has_grad) {
            c[h] = load4(t.acc_steps, q);
            u[h] = load4(t.updates, q);
            g[h] = load_grad4(t.grad, (b.grad_bf16 >> i) & 1u, q);
            m[h] = load4(t.m, q);
            v[h] = load4(t.v, q);
        }
        if (!b.opens) {
            prev[h] = load4(t.w_prev, q);
            dw[h] = load4(t.dist_w, q);
            dq[h] = load4(t.dist_q, q);
            codes_prev[h] = reinterpret_cast<const uint16_t*>(t.codes_prev)[q];
            byte[h] = t.scales_prev[q >> 3];
        }
    }
    if (has_grad) {
#pragma unroll
        for (int h = 0; h < H; ++h) {
            acc[h] = v4f{0.f, 0.f, 0.f, 0.f};
            if ((c[h].x | c[h].y | c[h].z | c[h].w) != 0) acc[h] = load4(t.g_acc, min(q0 + 64u * h, quads - 1u));
        }
    }
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const uint32_t q = q0 + 64u * h;
        const bool ok = q < quads;
        if (b.opens) {
            codes_prev[h] = rtn_codes4<FLOOR>(w[h], byte[h]);
            prev[h] = w[h];
            dw[h] = dq[h] = v4f{0.f, 0.f, 0.f, 0.f};
        }
        const v4f wq_prev = dequantize4(codes_prev[h], byte[h]);
        if (has_grad) {
            const bool held = (c[h].x | c[h].y | c[h].z | c[h].w) != 0;
            u[h] += 1;
            const bool uniform = uniform_updates(u[h]);
            StepScale k = step_scale(a, u[h].x, 1);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (!uniform && e > 0) k = step_scale(a, u[h][e], 1);
                const float gm = held ? __fdiv_rn(acc[h][e] + g[h][e], (float)(c[h][e] + 1)) : 0.0f + g[h][e];
                float we = w[h][e], me = m[h][e], ve = v[h][e];
                adamw_update(a, we, me, ve, gm, k);
                w[h][e] = we; m[h][e] = me; v[h][e] = ve;
            }
            if (ok) {
                store4(t.m, q, m[h]);
                store4(t.v, q, v[h]);
                store4(t.updates, q, u[h]);
                store4(t.w, q, w[h]);
                if (held) {
                    store4(t.g_acc, q, v4f{0.f, 0.f, 0.f, 0.f});
                    store4(t.acc_steps, q, v4i{0, 0, 0, 0});
                }
            }
        }
        const uint32_t p = rtn_codes4<FLOOR>(w[h], byte[h]);
        const v4f wq = dequantize4(p, byte[h]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            dw[h][e] = __fadd_rn(dw[h][e], __builtin_fabsf(__fsub_rn(w[h][e], prev[h][e])));
            dq[h][e] = __fadd_rn(dq[h][e], __builtin_fabsf(__fsub_rn(wq[e], wq_prev[e])));
        }
        if (ok) {
            store4(t.w_prev, q, w[h]);
            store4(t.dist_w, q, dw[h]);
            store4(t.dist_q, q, dq[h]);
            reinterpret_cast<uint16_t*>(t.codes_prev)[q] = (uint16_t)p;
            if ((threadIdx.x & 7) == 0) t.scales_prev[q >> 3] = (uint8_t)byte[h];
        }
    }
}

}  // namespace

namespace mxl {

// One launch of up to N tensors.
template <int N>
static hipError_t launch_adamw(const RampingAdamwParams* p, int count, hipStream_t st)
{
    AdamBatch<N> b{};
    b.h = hyper_of(p[0].lr, p[0].beta1, p[0].beta2, p[0].eps, p[0].weight_decay);
    const bool ramping = p[0].factor != nullptr;
    uint32_t blocks = 0;
    for (int i = 0; i < N; ++i) {
        b.end[i] = 0xFFFFFFFFu;
        if (i >= count) continue;
        const RampingAdamwParams& q = p[i];
        if ((q.factor != nullptr) != ramping) return hipErrorInvalidValue;
        b.t[i] = {q.w, q.grad, q.m, q.v, q.updates, q.g_acc, q.factor, q.acc_steps};
        b.quads[i] = q.count / 4;
        if (q.grad_bf16) b.grad_bf16 |= 1u << i;
        blocks += (uint32_t)((b.quads[i] + OPT_THREADS - 1) / OPT_THREADS);
        b.end[i] = blocks;
    }
    if (blocks == 0) return hipSuccess;
    if (ramping) hipLaunchKernelGGL((ramping_adamw_kernel<true, N>), dim3(blocks), dim3(OPT_THREADS), 0, st, b);
    else         hipLaunchKernelGGL((ramping_adamw_kernel<false, N>), dim3(blocks), dim3(OPT_THREADS), 0, st, b);
    return hipGetLastError();
}

hipError_t launch_ramping_adamw_batch(const RampingAdamwParams* p, int count, hipStream_t st)
{
    hipError_t e = hipSuccess;
    for (int at = 0; at < count && e == hipSuccess; at += ADAM_BATCH) {
        const int n = std::min(count - at, ADAM_BATCH);
        e = n == 1 ? launch_adamw<1>(p + at, 1, st) : launch_adamw<ADAM_BATCH>(p + at, n, st);
    }
    return e;
}

hipError_t launch_ramping_window_batch(const RampingWindowParams& p, const WindowTensor* tensors, const int64_t* counts,
                                       const bool* grad_bf16, int count, hipStream_t st)
{
    for (int at = 0; at < count; at += WINDOW_BATCH) {
        WindowBatch b{};
        b.h = hyper_of(p.lr, p.beta1, p.beta2, p.eps, p.weight_decay);
        b.opens = p.opens ? 1 : 0;
        const int n = count - at < WINDOW_BATCH ? count - at : WINDOW_BATCH;
        uint32_t blocks = 0;
        for (int i = 0; i < WINDOW_BATCH; ++i) {
            b.end[i] = 0xFFFFFFFFu;
            if (i >= n) continue;
            b.t[i] = tensors[at + i];
            b.quads[i] = (uint32_t)(counts[at + i] / 4);
            if (grad_bf16[at + i]) b.grad_bf16 |= 1u << i;
            blocks += (b.quads[i] + OPT_THREADS * WINDOW_QUADS - 1) / (OPT_THREADS * WINDOW_QUADS);
            b.end[i] = blocks;
        }
        if (p.floor_mode) hipLaunchKernelGGL(ramping_window_kernel<true>, dim3(blocks), dim3(OPT_THREADS), 0, st, b);
        else              hipLaunchKernelGGL(ramping_window_kernel<false>, dim3(blocks), dim3(OPT_THREADS), 0, st, b);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_ramping_adamw(const RampingAdamwParams& p, hipStream_t st) { return launch_ramping_adamw_batch(&p, 1, st); }

}  // namespace mxl
