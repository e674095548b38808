// Native host path of the Python front ends: one call per pass of a layer instead of a Python call per kernel.
// Host code only -- every quantizer and product is a launch of libmxfp4_hip.so (mx_launch.hpp); this file
// allocates, fills the launch arguments and carries the autograd graph.
//
// Why it is native: a forward + backward of one layer is 8 to 11 launches, and through Python each cost 8-12 us of
// argument handling next to 5-15 us of kernel for ViT-Tiny's sizes (270 us per layer, 110 us of it on the GPU).
#include <torch/extension.h>
#include <c10/hip/HIPGuard.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/mxfp4.h"
#include "mx_launch.hpp"

namespace {

using at::Tensor;
using OptTensor = std::optional<Tensor>;

// tensor ids of the six quantizers, numbered as in Eqs. 3-5
enum : uint32_t { Q1 = 1, Q2 = 2, Q3 = 3, Q4 = 4, Q5 = 5, Q6 = 6 };

// A refusal or a launch failure, with the C interface's code: binding.MxError in Python.
struct Status : std::runtime_error {
    std::string fn;
    int code, hip;
    Status(const char* f, int c, int h = 0) : std::runtime_error(std::string(f) + " failed: code " + std::to_string(c)), fn(f), code(c), hip(h) {}
};

PyObject* mx_error_class = nullptr;          // set once, when binding.py loads this module

// Sets the Python error of a Status; the caller holds the GIL.
void raise_in_python(const Status& s)
{
    if (mx_error_class == nullptr) {
        PyErr_SetString(PyExc_RuntimeError, s.what());
        return;
    }
    PyObject* e = PyObject_CallFunction(mx_error_class, "sii", s.fn.c_str(), s.code, s.hip);
    if (e == nullptr) return;                // the failure to make it is the error then
    PyErr_SetObject(mx_error_class, e);
    Py_DECREF(e);
}

void check(int code, const char* fn)
{
    if (code != MX_OK) throw Status(fn, code);
}

bool floor_of(int scale_mode, const char* fn)
{
    if (scale_mode != MX_SCALE_TRUNCFREE && scale_mode != MX_SCALE_FLOOR) throw Status(fn, MX_ERR_MODE);
    return scale_mode == MX_SCALE_FLOOR;
}

void check_hip(hipError_t e, const char* fn)
{
    if (e != hipSuccess) throw Status(fn, MX_ERR_HIP, (int)e);
}

bool is_bf16(const Tensor& t)
{
    TORCH_CHECK_TYPE(t.scalar_type() == at::kFloat || t.scalar_type() == at::kBFloat16,
                     "source must be float32 or bfloat16, got ", t.scalar_type());
    return t.scalar_type() == at::kBFloat16;
}

// Dense rows at a 16-byte aligned address, as the quantizers read them.
Tensor dense_source(const Tensor& t)
{
    Tensor c = t.contiguous();
    return (reinterpret_cast<uintptr_t>(c.data_ptr()) & 15) ? c.clone() : c;
}

int64_t round_up(int64_t v, int64_t to) { return (v + to - 1) / to * to; }

// Pieces of one device buffer, each 256-byte aligned.
struct Carver {
    int64_t used = 0;
    int64_t take(int64_t bytes)
    {
        const int64_t at = used;
        used += round_up(bytes, 256);
        return at;
    }
    int64_t codes(int64_t rows, int64_t cols) { return take(rows * (cols / 2)); }
    int64_t scales(int64_t rows, int64_t cols) { return take(rows * (cols / 32)); }
};

Tensor bytes_like(const Tensor& t, int64_t n) { return at::empty({n}, t.options().dtype(at::kByte)); }

struct Seed {
    uint64_t value = 0;
    const uint64_t* dev = nullptr;
};

Seed seed_of(int64_t value, const OptTensor& dev)
{
    Seed s{(uint64_t)value, nullptr};
    if (dev) {
        TORCH_CHECK_VALUE(dev->scalar_type() == at::kLong && dev->numel() == 1 && dev->is_cuda(),
                          "a device seed is a one-element int64 tensor on the GPU");
        s.dev = reinterpret_cast<const uint64_t*>(dev->data_ptr<int64_t>());
    }
    return s;
}

// One product C[m x n] = A . B^T into `out` (row pitch ldc); the workspace of a K split is not set.
mxl::GemmParams product_params(const uint8_t* a, const uint8_t* as, const uint8_t* b, const uint8_t* bs, int64_t m, int64_t n, int64_t k,
                               const Tensor& out, int64_t ldc, const float* bias, const char* fn)
{
    mxl::GemmParams p{};
    p.a_codes = a; p.a_scales = as; p.b_codes = b; p.b_scales = bs;
    p.m = m; p.n = n; p.k = k;
    p.c = out.data_ptr(); p.c_bf16 = is_bf16(out); p.ldc = ldc;
    p.bias = bias;
    check(mxl::check_gemm(p), fn);
    p.split_k = mxl::gemm_split_k(m, n, k);
    return p;
}

// Workspaces of the K splits of one product or of two that go to launch_gemm_pair: `given` where it is large enough, otherwise
// pieces of a buffer of the pass's own, returned to the allocator in stream order; `own` keeps it.  Products that run one after
// the other share a piece, so that a pass holds no more than the larger of the two needs.
void set_workspaces(mxl::GemmParams* w, mxl::GemmParams* x, const Tensor* given, const Tensor& like, Tensor& own, const char* fn)
{
    auto need = [&](mxl::GemmParams* p) -> int64_t {
        if (p == nullptr || p->split_k <= 1) return 0;
        const int64_t bytes = round_up((int64_t)p->split_k * p->m * p->n * 4, 256);
        if (given == nullptr || !given->defined() || (int64_t)given->nbytes() < (int64_t)p->split_k * p->m * p->n * 4) return bytes;
        p->workspace = given->data_ptr();
        return 0;
    };
    const int64_t nw = need(w), nx = need(x), behind = nw > 0 && nx > 0 && mxl::gemm_pair_fits_one_launch(*w, *x) ? nw : 0;
    if (nw > 0 || nx > 0) own = bytes_like(like, std::max(nw, behind + nx));
    if (nw > 0) w->workspace = own.data_ptr<uint8_t>();
    if (nx > 0) x->workspace = own.data_ptr<uint8_t>() + behind;
    for (mxl::GemmParams* p : {w, x})
        if (p != nullptr && p->split_k > 1 && (reinterpret_cast<uintptr_t>(p->workspace) & 255) != 0)
            throw Status(p == x ? "mx_linear_bwd_dx" : fn, MX_ERR_ALIGN);
}

void product(const uint8_t* a, const uint8_t* as, const uint8_t* b, const uint8_t* bs, int64_t m, int64_t n, int64_t k,
             const Tensor& out, int64_t ldc, const float* bias, hipStream_t st, const char* fn, const Tensor* workspace = nullptr)
{
    Tensor own;
    mxl::GemmParams p = product_params(a, as, b, bs, m, n, k, out, ldc, bias, fn);
    set_workspaces(&p, nullptr, workspace, out, own, fn);
    check_hip(mxl::launch_gemm(p, st), fn);
}

mxl::QuantRowsParams rows_job(const Tensor& src, int64_t rows, int64_t cols, uint8_t* codes, uint8_t* scales, bool floor_mode)
{
    mxl::QuantRowsParams q{};
    q.src = src.data_ptr(); q.bf16 = is_bf16(src);
    q.rows = rows; q.cols = cols; q.ld = cols;
    q.codes = codes; q.scales = scales;
    q.floor_mode = floor_mode;
    return q;
}

struct Layer {
    double beta;
    int update_ema;          // 0, 1, 2 as in mx_ema_weight_quant; used with a w_ema
    bool tetra, floor_mode;
};

void ema_rows(const Tensor& w, const Tensor& w_ema, const Layer& o, int64_t C, int64_t D, uint8_t* codes, uint8_t* scales, hipStream_t st)
{
    check_hip(mxl::launch_ema_quantize(rows_job(w, C, D, codes, scales, o.floor_mode), w_ema.data_ptr<float>(), (float)o.beta, o.update_ema, st),
              "mx_ema_weight_quant");
}

// The row and tile quantizers' launches behind their argument checks.
void launch_rows(const mxl::QuantRowsParams* q, int count, hipStream_t st, const mxl::WidenJob* widen)
{
    for (int j = 0; j < count; ++j) check(mxl::check_rows(q[j]), "mx_quantize");
    check_hip(mxl::launch_quantize_rows_batch(q, count, st, widen), "mx_quantize");
}

void launch_tiles(const mxl::QuantTileParams* q, int count, hipStream_t st, const mxl::WidenJob* widen = nullptr, bool finish_col_sums = true)
{
    const char* fn = count > 1 ? "mx_quantize_transposed_batch" : "mx_quantize_transposed";
    for (int j = 0; j < count; ++j) check(mxl::check_tile(q[j]), fn);
    check_hip(mxl::launch_quantize_tile_batch(q, count, st, widen, finish_col_sums), fn);
}

bool is_f32_or_bf16(at::ScalarType t) { return t == at::kFloat || t == at::kBFloat16; }

// FP32 bias: the tensor itself, a place in `base` that a quantizer launch widens bf16 into, or a converted copy.
const float* bias_source(const OptTensor& bias, Tensor& keep, uint8_t* place, mxl::WidenJob& widen)
{
    if (!bias) return nullptr;
    keep = dense_source(is_f32_or_bf16(bias->scalar_type()) ? *bias : bias->to(at::kFloat));
    if (!is_bf16(keep)) return keep.data_ptr<float>();
    widen.src = static_cast<const uint16_t*>(keep.data_ptr());
    widen.dst = reinterpret_cast<float*>(place);
    widen.count = (uint32_t)keep.numel();
    return widen.dst;
}

std::vector<int64_t> with_last(at::IntArrayRef sizes, int64_t last)
{
    std::vector<int64_t> s(sizes.begin(), sizes.end());
    s.back() = last;
    return s;
}

// Token rows of the packed operands: whole 32-row groups, and from 4096 rows on whole K steps (128) of the dW product,
// so that it runs on the main kernel.  Rows past N are zero: they change no group maximum and add nothing to dW.
int64_t padded_rows(int64_t N) { return round_up(N, N >= 4096 ? 128 : 32); }

// Whether work on the stream is being recorded into a graph.
bool is_capturing(hipStream_t st)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &status) != hipSuccess) {
        (void)hipGetLastError();                             // the launches report what is wrong with the stream
        return false;
    }
    return status == hipStreamCaptureStatusActive;
}

// Forward pass.  saved: null where no gradient will be asked for -- only the row codes are made then -- or
// receives the packed transposed operands [xtq | xts | wtq | wts] of the backward pass.
Tensor forward_pass(const Tensor& x_in, const Tensor& w_in, const OptTensor& bias, const OptTensor& w_ema, const Layer& o, const Seed& seed,
                    Tensor* saved)
{
    const Tensor x = dense_source(x_in), w = dense_source(w_in);
    const int64_t D = w.size(1), C = w.size(0), N = x.numel() / D;
    const int64_t Np = saved ? padded_rows(N) : N;
    hipStream_t st = c10::hip::getCurrentHIPStream(x.get_device()).stream();

    const bool captured = !saved && D > 256 && D <= 512 && is_capturing(st);         // where the rule asks for it
    if (!saved && !w_ema && mxl::linear_fits_one_launch(N, C, D, bias && bias->scalar_type() == at::kBFloat16, captured)) {
        Tensor b, y = at::empty(with_last(x_in.sizes(), C), x.options());
        if (bias) b = dense_source(is_f32_or_bf16(bias->scalar_type()) ? *bias : bias->to(at::kFloat));
        const mxl::QuantizedLinearParams p{x.data_ptr(), w.data_ptr(), bias ? b.data_ptr() : nullptr, is_bf16(x), is_bf16(w), bias && is_bf16(b), o.floor_mode,
                                           N, C, D, y.data_ptr(), is_bf16(y)};
        check_hip(mxl::launch_quantized_linear(p, st), "mx_linear_fwd");
        return y;
    }

    Carver t;
    const int64_t o_xq = t.codes(Np, D), o_xs = t.scales(Np, D), o_wq = t.codes(C, D), o_ws = t.scales(C, D), o_b = t.take(C * 4);
    Tensor row = bytes_like(x, t.used), keep;
    uint8_t* r = row.data_ptr<uint8_t>();
    mxl::WidenJob widen;
    const float* b32 = bias_source(bias, keep, r + o_b, widen);

    if (!saved) {
        mxl::QuantRowsParams q[2] = {rows_job(x, N, D, r + o_xq, r + o_xs, o.floor_mode), rows_job(w, C, D, r + o_wq, r + o_ws, o.floor_mode)};
        launch_rows(q, w_ema ? 1 : 2, st, &widen);
        if (w_ema) ema_rows(w, *w_ema, o, C, D, r + o_wq, r + o_ws, st);
    } else {
        Carver v;
        const int64_t o_xtq = v.codes(D, Np), o_xts = v.scales(D, Np), o_wtq = v.codes(D, C), o_wts = v.scales(D, C);
        *saved = bytes_like(x, v.used);
        uint8_t* s = saved->data_ptr<uint8_t>();
        mxl::QuantTileParams q[2] = {};
        auto job = [&](mxl::QuantTileParams& j, const Tensor& src, int64_t rows, int64_t src_rows, uint32_t tid_t, uint32_t tid_row) {
            j.src = src.data_ptr(); j.bf16 = is_bf16(src);
            j.rows = rows; j.src_rows = src_rows; j.cols = D; j.ld = D;
            j.sr_t = o.tetra; j.tensor_id_t = tid_t; j.pre_quant = o.tetra; j.tensor_id_row = tid_row;
            j.floor_mode = o.floor_mode; j.seed = seed.value; j.seed_dev = seed.dev;
        };
        job(q[0], x, Np, N, Q6, Q1);
        q[0].codes_t = s + o_xtq; q[0].scales_t = s + o_xts; q[0].codes_row = r + o_xq; q[0].scales_row = r + o_xs;
        job(q[1], w, C, C, Q4, Q2);
        q[1].codes_t = s + o_wtq; q[1].scales_t = s + o_wts; q[1].codes_row = r + o_wq; q[1].scales_row = r + o_ws;
        launch_tiles(q, w_ema ? 1 : 2, st, &widen);
        if (w_ema) {
            ema_rows(w, *w_ema, o, C, D, r + o_wq, r + o_ws, st);
            q[1].codes_row = q[1].scales_row = nullptr;
            if (o.tetra) {                                   // double quantization of the codes the forward product uses
                q[1].src = nullptr; q[1].bf16 = false;
                q[1].row_codes_in = r + o_wq; q[1].row_scales_in = r + o_ws;
            }
            launch_tiles(q + 1, 1, st);
        }
    }
    Tensor y = at::empty(with_last(x_in.sizes(), C), x.options());
    product(r + o_xq, r + o_xs, r + o_wq, r + o_ws, N, C, D, y, C, b32, st, bias ? "mx_linear_fwd_bias" : "mx_linear_fwd");
    return y;
}

struct MxLinearFn : torch::autograd::Function<MxLinearFn> {
    static Tensor forward(torch::autograd::AutogradContext* ctx, const Tensor& x, const Tensor& w, const OptTensor& bias, const OptTensor& w_ema,
                          int64_t update_ema, double beta, bool tetra, bool floor_mode, int64_t seed, const OptTensor& seed_dev)
    {
        at::AutoDispatchBelowADInplaceOrView guard;
        Tensor saved;
        Tensor y = forward_pass(x, w, bias, w_ema, Layer{beta, (int)update_ema, tetra, floor_mode}, seed_of(seed, seed_dev), &saved);
        torch::autograd::variable_list keep{saved};
        if (seed_dev) keep.push_back(*seed_dev);
        ctx->save_for_backward(keep);
        ctx->saved_data["shape"] = x.sizes().vec();
        ctx->saved_data["meta"] = std::vector<int64_t>{w.size(0), w.size(1), (int64_t)tetra, (int64_t)floor_mode, seed,
                                                       (int64_t)w.scalar_type(), bias ? (int64_t)bias->scalar_type() : -1};
        return y;
    }

    // The engine carries a Python error to the caller of backward() as it is, any other exception as a RuntimeError.
    static torch::autograd::variable_list backward(torch::autograd::AutogradContext* ctx, torch::autograd::variable_list grads)
    {
        try {
            return backward_pass(ctx, grads);
        } catch (const Status& s) {
            py::gil_scoped_acquire gil;
            raise_in_python(s);
            python_error e;
            e.persist();
            throw e;
        }
    }

    static torch::autograd::variable_list backward_pass(torch::autograd::AutogradContext* ctx, const torch::autograd::variable_list& grads)
    {
        at::AutoDispatchBelowADInplaceOrView guard;
        const auto keep = ctx->get_saved_variables();
        const auto shape = ctx->saved_data["shape"].toIntVector(), meta = ctx->saved_data["meta"].toIntVector();
        const int64_t C = meta[0], D = meta[1], seed_value = meta[4];
        const bool tetra = meta[2] != 0, floor_mode = meta[3] != 0, has_bias = meta[6] >= 0;
        const bool want_dx = ctx->needs_input_grad(0), want_dw = ctx->needs_input_grad(1), want_db = has_bias && ctx->needs_input_grad(2);
        const Seed seed = seed_of(seed_value, keep.size() > 1 ? OptTensor(keep[1]) : OptTensor());

        const Tensor dy = dense_source(grads[0]);
        c10::hip::HIPGuard device((c10::DeviceIndex)dy.get_device());
        const int64_t N = dy.numel() / C, Np = padded_rows(N);
        hipStream_t st = c10::hip::getCurrentHIPStream(dy.get_device()).stream();
        Carver v;
        const int64_t o_xtq = v.codes(D, Np), o_xts = v.scales(D, Np), o_wtq = v.codes(D, C), o_wts = v.scales(D, C);
        // what the forward pass saved may have gone through a program's pack and unpack hooks
        if (keep[0].scalar_type() != at::kByte || keep[0].numel() != v.used || !keep[0].is_contiguous() || keep[0].get_device() != dy.get_device())
            throw Status("mx_linear_bwd", MX_ERR_SHAPE);
        const uint8_t* s = keep[0].data_ptr<uint8_t>();

        Carver t;
        const int64_t o_q = t.codes(Np, C), o_s = t.scales(Np, C), o_tq = t.codes(C, Np), o_ts = t.scales(C, Np);
        const int64_t o_cs = t.take(want_db ? (int64_t)mxl::column_sum_workspace_bytes(Np, C) : 0);
        Tensor packed = bytes_like(dy, t.used);
        uint8_t* p = packed.data_ptr<uint8_t>();

        Tensor dx, dw, db;
        mxl::ColumnSumTail tail{};
        if (want_dw || want_db) {
            mxl::QuantTileParams q{};
            q.src = dy.data_ptr(); q.bf16 = is_bf16(dy);
            q.rows = Np; q.src_rows = N; q.cols = C; q.ld = C;
            q.codes_t = p + o_tq; q.scales_t = p + o_ts; q.sr_t = tetra; q.tensor_id_t = Q5;
            q.codes_row = want_dx ? p + o_q : nullptr; q.scales_row = want_dx ? p + o_s : nullptr;
            q.sr_row = tetra; q.tensor_id_row = Q3;
            q.floor_mode = floor_mode; q.seed = seed.value; q.seed_dev = seed.dev;
            if (want_db) {
                const at::ScalarType type = (at::ScalarType)meta[6];
                db = at::empty({C}, dy.options().dtype(is_f32_or_bf16(type) ? type : at::kFloat));
                q.col_sums = db.data_ptr(); q.col_sums_bf16 = is_bf16(db);
                q.col_sum_workspace = reinterpret_cast<float*>(p + o_cs);
                tail = mxl::column_sum_tail(q);
            }
            launch_tiles(&q, 1, st, nullptr, false);
        } else if (want_dx && !seed.dev) {
            mxl::QuantRowsParams q = rows_job(dy, N, C, p + o_q, p + o_s, floor_mode);
            q.sr = tetra; q.seed = seed.value; q.tensor_id = Q3;
            check(mxl::check_rows(q), "mx_quantize");
            check_hip(mxl::launch_quantize_rows(q, st), "mx_quantize");
        } else if (want_dx) {                                // the row quantizer takes its seed by value only
            mxl::QuantTileParams q{};
            q.src = dy.data_ptr(); q.bf16 = is_bf16(dy);
            q.rows = Np; q.src_rows = N; q.cols = C; q.ld = C;
            q.codes_t = p + o_tq; q.scales_t = p + o_ts; q.sr_t = tetra; q.tensor_id_t = Q5;
            q.codes_row = p + o_q; q.scales_row = p + o_s; q.sr_row = tetra; q.tensor_id_row = Q3;
            q.floor_mode = floor_mode; q.seed_dev = seed.dev;
            launch_tiles(&q, 1, st);
        }
        const mxl::ColumnSumTail* sums = want_db ? &tail : nullptr;
        mxl::GemmParams px, pw;
        Tensor own;
        if (want_dx) {
            dx = at::empty(shape, dy.options());
            px = product_params(p + o_q, p + o_s, s + o_wtq, s + o_wts, N, D, C, dx, D, nullptr, "mx_linear_bwd_dx");
        }
        if (want_dw) {
            dw = at::empty({C, D}, dy.options().dtype((at::ScalarType)meta[5]));
            pw = product_params(p + o_tq, p + o_ts, s + o_xtq, s + o_xts, C, D, Np, dw, D, nullptr, "mx_linear_bwd_dw");
        }
        set_workspaces(want_dw ? &pw : nullptr, want_dx ? &px : nullptr, nullptr, dy, own, "mx_linear_bwd_dw");
        if (want_dx && want_dw) {
            check_hip(mxl::launch_gemm_pair(pw, px, st, sums), "mx_linear_bwd_dw");
        } else if (want_dx) {
            check_hip(mxl::launch_gemm(px, st), "mx_linear_bwd_dx");
        } else if (want_dw) {
            check_hip(mxl::launch_gemm(pw, st, sums), "mx_linear_bwd_dw");
        }
        if (!want_dw && want_db) {
            check_hip(mxl::launch_column_sum_finish(tail, st), "mx_quantize_transposed_batch");
        }
        if (want_db) db = db.to((at::ScalarType)meta[6]);
        return {dx, dw, db, Tensor(), Tensor(), Tensor(), Tensor(), Tensor(), Tensor(), Tensor()};
    }
};

// What the pass relies on, looked at before any of it runs (and before the device, so that it can be tested without one).
// weight is a parameter that a program may replace: its sizes are looked at on every call.
void check_layer(const Tensor& x, const Tensor& w, const OptTensor& bias, const OptTensor& w_ema, int64_t update_ema, double beta, const OptTensor& seed_dev)
{
    // without a gradient to record the pass goes past the autograd node, which would refuse a tangent
    for (const Tensor* t : {&x, &w, bias ? &*bias : &x})
        TORCH_CHECK_NOT_IMPLEMENTED(!t->_fw_grad(0).defined(), "MxLinear has no forward-mode derivative");
    TORCH_CHECK(w.dim() == 2 && x.dim() >= 1 && x.size(-1) == w.size(1), "input of ", w.size(1), " features expected, got ", x.sizes());
    TORCH_CHECK(!bias || bias->numel() == w.size(0), "bias must have ", w.size(0), " values");
    if (x.numel() == 0 || w.numel() == 0 || w.size(0) % 32 != 0 || w.size(1) % 32 != 0) throw Status("mx_quantize_transposed", MX_ERR_SHAPE);
    if (w_ema) {
        TORCH_CHECK_VALUE(w_ema->scalar_type() == at::kFloat && w_ema->is_contiguous() && w_ema->sizes() == w.sizes(),
                          "w_ema must be float32 with the shape and strides of w");
        mxl::QuantRowsParams q{};
        q.rows = w.size(0); q.cols = q.ld = w.size(1);
        check(mxl::check_ema(q, w_ema->data_ptr<float>(), (float)beta, (int)update_ema), "mx_ema_weight_quant");
    }
    TORCH_CHECK(x.is_cuda(), "MxLinear runs on the GPU");
    auto there = [&](const Tensor& t) { return t.get_device() == x.get_device(); };
    TORCH_CHECK(there(w) && (!bias || there(*bias)) && (!w_ema || there(*w_ema)) && (!seed_dev || there(*seed_dev)),
                "MxLinear: x, weight, bias, moving average and seed must be on one GPU");
}

Tensor linear(const Tensor& x, const Tensor& w, const OptTensor& bias, const OptTensor& w_ema, int64_t update_ema, double beta, bool tetra,
              int scale_mode, uint64_t seed, const OptTensor& seed_dev)
{
    const bool floor_mode = floor_of(scale_mode, "mx_quantize_transposed");
    check_layer(x, w, bias, w_ema, update_ema, beta, seed_dev);
    c10::hip::HIPGuard device((c10::DeviceIndex)x.get_device());
    const bool grad = at::GradMode::is_enabled() && (x.requires_grad() || w.requires_grad() || (bias && bias->requires_grad()));
    if (!grad) {
        at::AutoDispatchBelowADInplaceOrView guard;
        return forward_pass(x, w, bias, w_ema, Layer{beta, (int)update_ema, tetra, floor_mode}, Seed{}, nullptr);
    }
    return MxLinearFn::apply(x, w, bias, w_ema, update_ema, beta, tetra, floor_mode, (int64_t)seed, seed_dev);
}

// ---- MxLinearStep: the same passes on the caller's buffers ----

uint8_t* u8(const Tensor& t) { return t.data_ptr<uint8_t>(); }

void check_source(const Tensor& t, int64_t rows, int64_t cols, const char* name)
{
    TORCH_CHECK_VALUE(t.dim() == 2 && t.size(0) == rows && t.size(1) == cols && t.stride(1) == 1, name, " must be a [", rows, ", ", cols,
                      "] matrix with unit column stride");
    const bool bf16 = is_bf16(t);
    if (t.stride(0) < cols) throw Status("mx_quantize_transposed", MX_ERR_SHAPE);
    if ((reinterpret_cast<uintptr_t>(t.data_ptr()) & 15) != 0 || t.stride(0) % (bf16 ? 8 : 4) != 0) throw Status("mx_quantize_transposed", MX_ERR_ALIGN);
    TORCH_CHECK_VALUE(t.is_cuda(), name, " must be on the GPU");
}

mxl::QuantTileParams tile_job(const Tensor& src, int64_t rows, int64_t cols, const std::vector<Tensor>& out, bool sr_t, uint32_t tid_t,
                              bool pre, bool sr_row, uint32_t tid_row, bool floor_mode, const Seed& seed)
{
    mxl::QuantTileParams j{};
    j.src = src.data_ptr(); j.bf16 = is_bf16(src);
    j.rows = rows; j.cols = cols; j.ld = src.stride(0);
    j.codes_row = u8(out[0]); j.scales_row = u8(out[1]); j.codes_t = u8(out[2]); j.scales_t = u8(out[3]);
    j.sr_t = sr_t; j.tensor_id_t = tid_t; j.pre_quant = pre; j.sr_row = sr_row; j.tensor_id_row = tid_row;
    j.floor_mode = floor_mode; j.seed = seed.value; j.seed_dev = seed.dev;
    return j;
}

// xb, wb: (row codes, row scales, transposed codes, transposed scales) of X and W.
void step_forward(const Tensor& X, const Tensor& W, int64_t N, int64_t D, int64_t C, uint64_t seed_value, const OptTensor& seed_dev,
                  const std::vector<Tensor>& xb, const std::vector<Tensor>& wb, const Tensor& y, const Tensor& workspace, int scale_mode)
{
    const bool floor_mode = floor_of(scale_mode, "mx_quantize_transposed");
    check_source(X, N, D, "X");
    check_source(W, C, D, "W");
    const Seed seed = seed_of((int64_t)seed_value, seed_dev);
    hipStream_t st = c10::hip::getCurrentHIPStream().stream();
    const mxl::QuantTileParams q[2] = {tile_job(X, N, D, xb, true, Q6, true, false, Q1, floor_mode, seed),
                                       tile_job(W, C, D, wb, true, Q4, true, false, Q2, floor_mode, seed)};
    launch_tiles(q, 2, st);
    product(u8(xb[0]), u8(xb[1]), u8(wb[0]), u8(wb[1]), N, C, D, y, y.stride(0), nullptr, st, "mx_linear_fwd", &workspace);
}

void step_backward(const Tensor& dY, int64_t N, int64_t D, int64_t C, uint64_t seed_value, const OptTensor& seed_dev, const std::vector<Tensor>& dyb,
                   const std::vector<Tensor>& wt, const std::vector<Tensor>& xt, const Tensor& dx, const Tensor& dw, const Tensor& workspace,
                   int scale_mode)
{
    const bool floor_mode = floor_of(scale_mode, "mx_quantize_transposed");
    check_source(dY, N, C, "dY");
    hipStream_t st = c10::hip::getCurrentHIPStream().stream();
    const mxl::QuantTileParams q = tile_job(dY, N, C, dyb, true, Q5, false, true, Q3, floor_mode, seed_of((int64_t)seed_value, seed_dev));
    launch_tiles(&q, 1, st);
    mxl::GemmParams px = product_params(u8(dyb[0]), u8(dyb[1]), u8(wt[0]), u8(wt[1]), N, D, C, dx, dx.stride(0), nullptr, "mx_linear_bwd_dx");
    mxl::GemmParams pw = product_params(u8(dyb[2]), u8(dyb[3]), u8(xt[0]), u8(xt[1]), C, D, N, dw, dw.stride(0), nullptr, "mx_linear_bwd_dw");
    Tensor own;
    set_workspaces(&pw, &px, &workspace, dY, own, "mx_linear_bwd_dw");
    check_hip(mxl::launch_gemm_pair(pw, px, st), "mx_linear_bwd_dw");
}

// ---- QRampingAdamW: one call per parameter group ----

// A tensor of an optimizer state dict.
const Tensor& state_tensor(PyObject* state, PyObject* key)
{
    PyObject* v = PyDict_GetItem(state, key);               // borrowed
    TORCH_CHECK(v != nullptr && THPVariable_Check(v), "optimizer state is incomplete");
    return THPVariable_Unpack(v);
}

template <typename T>
T* checked(const Tensor& t, int64_t count, at::ScalarType type, const char* what, int device)
{
    TORCH_CHECK_VALUE(t.numel() == count && t.scalar_type() == type && t.is_contiguous(), what, ": a contiguous ", type, " tensor of ", count, " values expected");
    if ((reinterpret_cast<uintptr_t>(t.data_ptr()) & 15) != 0) throw Status("mx_ramping_adamw_step", MX_ERR_ALIGN);
    TORCH_CHECK(t.get_device() == device, what, ": not on the parameter's device");
    return reinterpret_cast<T*>(t.data_ptr());
}

// mode 0: plain AdamW, 1: with amplification factors, 2: a step inside a detection window (`opens`: its first).
// params and states are parallel lists; a parameter without a gradient is skipped (mode 2: only tracked).
void ramping_step(const py::list& params, const py::list& states, int mode, bool opens, int scale_mode, float lr, float beta1, float beta2,
                  float eps, float weight_decay)
{
    const bool floor_mode = mode == 2 && floor_of(scale_mode, "mx_quantize");       // used inside a window only
    static PyObject *k_m = PyUnicode_InternFromString("m"), *k_v = PyUnicode_InternFromString("v"), *k_u = PyUnicode_InternFromString("updates"),
                    *k_acc = PyUnicode_InternFromString("g_acc"), *k_steps = PyUnicode_InternFromString("acc_steps"),
                    *k_factor = PyUnicode_InternFromString("factor"), *k_prev = PyUnicode_InternFromString("w_prev"),
                    *k_dw = PyUnicode_InternFromString("dist_w"), *k_dq = PyUnicode_InternFromString("dist_q"),
                    *k_codes = PyUnicode_InternFromString("codes_prev"), *k_scales = PyUnicode_InternFromString("scales_prev");
    const Py_ssize_t n = PyList_GET_SIZE(params.ptr());
    TORCH_CHECK(PyList_GET_SIZE(states.ptr()) == n, "one state per parameter");
    // written so that NaN fails
    if (!(lr >= 0.0f && beta1 > 0.0f && beta1 < 1.0f && beta2 > 0.0f && beta2 < 1.0f && eps >= 0.0f && weight_decay >= 0.0f))
        throw Status("mx_ramping_adamw_step", MX_ERR_MODE);
    // one batch per device, in order
    std::vector<mxl::RampingAdamwParams> adam;
    std::vector<mxl::WindowTensor> window;
    std::vector<int64_t> counts;
    std::vector<Tensor> keep;                                // gradients made contiguous here live until the launch is enqueued
    std::unique_ptr<bool[]> bf16(new bool[n > 0 ? n : 1]);
    int device = -1;
    auto flush = [&]() {
        if (device < 0) return;
        c10::hip::HIPGuard guard((c10::DeviceIndex)device);
        hipStream_t st = c10::hip::getCurrentHIPStream((c10::DeviceIndex)device).stream();
        if (mode == 2) {
            const mxl::RampingWindowParams p{lr, beta1, beta2, eps, weight_decay, opens, floor_mode};
            check_hip(mxl::launch_ramping_window_batch(p, window.data(), counts.data(), bf16.get(), (int)window.size(), st), "mx_ramping_adamw_step");
        } else {
            check_hip(mxl::launch_ramping_adamw_batch(adam.data(), (int)adam.size(), st), "mx_ramping_adamw_step");
        }
        adam.clear(); window.clear(); counts.clear(); keep.clear();
    };
    for (Py_ssize_t i = 0; i < n; ++i) {
        PyObject* pp = PyList_GET_ITEM(params.ptr(), i);
        TORCH_CHECK(THPVariable_Check(pp), "parameters must be tensors");
        const Tensor& p = THPVariable_Unpack(pp);
        PyObject* st = PyList_GET_ITEM(states.ptr(), i);
        TORCH_CHECK(PyDict_Check(st), "states must be dicts");
        Tensor grad = p.grad();
        if (!grad.defined() && mode != 2) continue;
        if (p.get_device() != device) { flush(); device = p.get_device(); }
        // a group added later has not passed the constructor's checks
        const int64_t count = p.numel();
        if (mode == 2 && (p.dim() != 2 || p.size(1) % 32 != 0)) throw Status("mx_quantize", MX_ERR_SHAPE);
        if (count <= 0 || count % 4 != 0) throw Status("mx_ramping_adamw_step", MX_ERR_SHAPE);
        float* w = checked<float>(p, count, at::kFloat, "parameter", device);
        bool gb = false;
        if (grad.defined()) {
            TORCH_CHECK_VALUE(grad.sizes() == p.sizes(), "shape mismatch");
            gb = is_bf16(grad);
            grad = grad.contiguous();
            if ((reinterpret_cast<uintptr_t>(grad.data_ptr()) & (gb ? 7 : 15)) != 0) throw Status("mx_ramping_adamw_step", MX_ERR_ALIGN);
            TORCH_CHECK(grad.get_device() == device, "gradient: not on the parameter's device");
            keep.push_back(grad);
        }
        auto f32 = [&](PyObject* k) { return checked<float>(state_tensor(st, k), count, at::kFloat, "state", device); };
        auto i32 = [&](PyObject* k) { return checked<int32_t>(state_tensor(st, k), count, at::kInt, "state", device); };
        TORCH_CHECK(p.is_cuda(), "the optimizer's kernels run on the GPU");
        if (mode == 2) {
            auto u8s = [&](PyObject* k, int64_t per) { return checked<uint8_t>(state_tensor(st, k), count / per, at::kByte, "state", device); };
            bf16[window.size()] = gb;
            window.push_back({w, grad.defined() ? grad.data_ptr() : nullptr, f32(k_m), f32(k_v), i32(k_u), f32(k_acc), i32(k_steps), f32(k_prev),
                              f32(k_dw), f32(k_dq), u8s(k_codes, 2), u8s(k_scales, 32)});
            counts.push_back(count);
        } else {
            mxl::RampingAdamwParams a{};
            a.w = w; a.grad = grad.data_ptr(); a.grad_bf16 = gb; a.count = count;
            a.m = f32(k_m); a.v = f32(k_v); a.updates = i32(k_u);
            if (mode == 1) { a.g_acc = f32(k_acc); a.acc_steps = i32(k_steps); a.factor = i32(k_factor); }
            a.lr = lr; a.beta1 = beta1; a.beta2 = beta2; a.eps = eps; a.weight_decay = weight_decay;
            adam.push_back(a);
        }
    }
    flush();
}

}  // namespace

PYBIND11_MODULE(_mx_torch, m)
{
    py::register_local_exception_translator([](std::exception_ptr p) {
        try {
            if (p) std::rethrow_exception(p);
        } catch (const Status& s) {
            raise_in_python(s);
        }
    });
    m.def("set_error_class", [](py::object cls) {            // keeps the class for the life of the process
        Py_XDECREF(mx_error_class);
        mx_error_class = cls.release().ptr();
    });
    m.def("linear", &linear, py::call_guard<py::gil_scoped_release>());
    m.def("linear_fits_one_launch", &mxl::linear_fits_one_launch);           // the rules, for tests
    m.def("gemm_kernel_name", &mxl::gemm_kernel_name);
    m.def("tile_workgroups", &mxl::tile_workgroups);
    m.def("step_forward", &step_forward, py::call_guard<py::gil_scoped_release>());
    m.def("ramping_step", &ramping_step);
    m.def("step_backward", &step_backward, py::call_guard<py::gil_scoped_release>());
}
