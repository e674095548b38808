"""torch.autograd / nn.Module front end of the MXFP4 linear layer: the forward and backward of Eqs. 3-5
(Sec. 3.3).  Plumbing only -- the pass itself is one native call (csrc/mx_torch.cpp), every quantizer and
every product in it a kernel of the HIP library; what is saved for the backward pass is the packed 4-bit
operands, not the activations.  Where no gradient will be asked for (torch.no_grad(), or nothing requires
one) only the row codes are made, which is all the forward product reads."""
import itertools

import torch

from . import binding as B

TETRAJET, MICROSCALING = "tetrajet", "microscaling"

# Layers are numbered in the order they are constructed; the number goes into every layer's Philox key
# so that two layers never round with the same random numbers (see MxLinear).
_layer_ids = itertools.count()


class _TracedLinear(torch.autograd.Function):
    """The pass as torch.jit.trace records it: one call of this function, made again on every replay.  The native call
    itself would leave nothing but its allocations in a trace, because its kernels are launched past the dispatcher."""

    @staticmethod
    def forward(ctx, x, weight, bias, mod, seed, seed_dev):
        with torch.enable_grad():
            ctx.inputs = [None if t is None else t.detach().requires_grad_(need)
                          for t, need in zip((x, weight, bias), ctx.needs_input_grad)]
            ctx.y = mod._pass(*ctx.inputs, seed, seed_dev)
        return ctx.y.detach()

    @staticmethod
    def backward(ctx, dy):
        grads = iter(torch.autograd.grad(ctx.y, [t for t, need in zip(ctx.inputs, ctx.needs_input_grad) if need], dy, retain_graph=True))
        return tuple(next(grads) if need else None for need in ctx.needs_input_grad)


class MxLinear(torch.nn.Module):
    """y = x W^T (+ bias) with the three products in MXFP4 (Eqs. 3-5).

    in_features and out_features must be multiples of 32; the token count (product of the leading
    dimensions of x) is padded with zero rows to whole groups of 32 inside the quantizer.  x and weight are float32 or
    bfloat16.  flow="tetrajet": deterministic forward quantizers, stochastic backward quantizers,
    double quantization (Sec. 3.3); flow="microscaling": Eqs. 6-7 (all deterministic, the backward
    operands quantized from the full-precision tensors).  qema=True takes the forward weight codes
    from Q-EMA (Sec. 5); the moving average advances once per training-mode forward.

    Stochastic rounding streams.  The 64-bit Philox key of a forward call and of its backward is
    (seed & 0xFFFF) << 48 | (layer_id & 0xFFFF) << 32 | number of forward calls so far.  layer_id
    defaults to the layer's position in the order of construction in this process, so the layers of a
    model draw independent numbers (the unbiasedness argument of Sec. 3.4 needs the rounding of dY in
    one layer to be independent of the rounding that produced it in the next); pass layer_id to fix
    it, e.g. to reproduce a run with a different construction order.  device_seed=True keeps the key in
    device memory and advances it with a kernel, so that a forward + backward recorded into a graph
    rounds with new numbers on every replay (same values as the host-side key, call for call); each
    forward call keeps its own copy of the key for its backward, so several forwards may precede the
    first backward (micro-batches, a module used twice).
    """

    def __init__(self, in_features, out_features, bias=True, device="cuda", dtype=torch.float32,
                 flow=TETRAJET, scale_mode=B.SCALE_TRUNCFREE, qema=False, beta=0.998, seed=0, device_seed=False,
                 layer_id=None):
        super().__init__()
        if in_features % 32 or out_features % 32:
            raise ValueError("in_features and out_features must be multiples of 32")
        if flow not in (TETRAJET, MICROSCALING):
            raise ValueError("flow must be 'tetrajet' or 'microscaling'")
        self.in_features, self.out_features = in_features, out_features
        self.flow, self.scale_mode, self.qema, self.beta, self.seed = flow, scale_mode, qema, beta, int(seed)
        self.weight = torch.nn.Parameter(torch.empty((out_features, in_features), device=device, dtype=dtype))
        self.bias = torch.nn.Parameter(torch.zeros(out_features, device=device, dtype=dtype)) if bias else None
        torch.nn.init.trunc_normal_(self.weight, std=0.02)
        self.register_buffer("w_ema", torch.zeros((out_features, in_features), device=device, dtype=torch.float32)
                             if qema else None)
        self.calls = 0                     # forward calls so far (host-side: reading it must not synchronize)
        self.layer_id = next(_layer_ids) if layer_id is None else int(layer_id)
        self.key_high = ((self.seed & 0xFFFF) << 16) | (self.layer_id & 0xFFFF)   # upper 32 bits of the Philox key
        start = ((self.key_high << 32) - 1) & 0xFFFFFFFFFFFFFFFF                 # one before the first key, as a 64-bit word
        self.register_buffer("seed_state", torch.tensor([start - (1 << 64) if start >> 63 else start], dtype=torch.int64,
                                                        device=device) if device_seed else None)
        self._ema_started = False

    def _pass(self, x, weight, bias, seed, seed_dev):
        """The native call.  The call's key is seed, or the word in seed_dev where that is a tensor."""
        w_ema, update = None, 0
        if self.qema:                       # 2 starts the moving average from the weight, 1 advances it, 0 leaves it
            w_ema, update = self.w_ema, 2 if not self._ema_started else 1 if self.training else 0
            if w_ema is None:
                raise ValueError("Q-EMA needs the buffer w_ema, which the layer was made without")
        y = B.host().linear(x, weight, bias, w_ema, update, self.beta, self.flow == TETRAJET, self.scale_mode, seed, seed_dev)
        if update == 2:                     # not before: a refused call has started nothing
            self._ema_started = True
        return y

    def forward(self, x):
        seed_dev = None
        if self.seed_state is not None:
            # the word the kernels read: this call's own copy, which its backward pass reads too, so
            # that later forward calls (which advance seed_state) do not change it
            seed, seed_dev = 0, self.seed_state.add_(1).clone()
        else:
            seed = (self.key_high << 32) + (self.calls & 0xFFFFFFFF)
        self.calls += 1
        if torch.jit.is_tracing():
            return _TracedLinear.apply(x, self.weight, self.bias, self, seed, seed_dev)
        return self._pass(x, self.weight, self.bias, seed, seed_dev)
