"""Q-Ramping as a torch optimizer (Algorithm 2, Sec. 6): the schedule of the algorithm around the
library's kernels.  Plumbing only: every array operation is one of the library's kernels, which take the tensors
of a parameter group many at a time.

Every t_update steps a detection window of t0 steps opens.  Inside it the quantized weights take plain
AdamW steps (amplification factor 1 for every element) and the trajectory lengths dist_W, dist_Q of
Sec. 6.1 are accumulated from the weight before the window's first step to the weight after its last
one (t0 differences).  When the window closes, N_w = min(k2 * floor(R_w / k1) + 1, n_max) is computed
per element and used until the next window: an element then accumulates its gradient over N_w steps
and takes one AdamW step at N_w times the learning rate on the mean.  Parameters that are not
quantized take plain AdamW steps throughout.

Readings of the paper: the calibration steps of OscillationDetection are the training steps themselves;
w_Q is the forward quantizer's value of the master weight (1x32 groups along the input dimension, round
to nearest); gradients an element still holds when a window opens are applied at that step (their mean,
as one update).  t0 = 30 is the paper's value; t_update and n_max are not printed and must be chosen.
"""
import torch

from . import binding as B


class QRampingAdamW(torch.optim.Optimizer):
    """quantized: the master weights of MXFP4 layers (float32, [out, in] with `in` a multiple of 32);
    others: every other parameter (float32).  step() reads p.grad of each."""

    def __init__(self, quantized, others=(), lr=1e-3, betas=(0.9, 0.999), eps=1e-8, weight_decay=0.01,
                 k1=16.0, k2=5, n_max=16, t0=30, t_update=1000, scale_mode=B.SCALE_TRUNCFREE):
        if not 0 < t0 < t_update:
            raise ValueError("need 0 < t0 < t_update (Algorithm 2: T0 << T_update)")
        if n_max < 1 or k2 < 0 or not k1 > 0:
            raise ValueError("need n_max >= 1, k2 >= 0, k1 > 0")
        groups = [{"params": list(quantized), "quantized": True}, {"params": list(others), "quantized": False}]
        for g in groups:
            for p in g["params"]:
                if p.dtype != torch.float32 or not p.is_contiguous():
                    raise ValueError("parameters must be contiguous float32 (master weights)")
                if p.numel() % 4:
                    raise ValueError("the optimizer kernel takes arrays whose length is a multiple of 4")
                if g["quantized"] and (p.dim() != 2 or p.shape[1] % 32):
                    raise ValueError("a quantized weight is [out, in] with `in` a multiple of 32")
        defaults = dict(lr=lr, betas=betas, eps=eps, weight_decay=weight_decay, k1=k1, k2=k2, n_max=n_max,
                        t0=t0, t_update=t_update, scale_mode=scale_mode, steps_done=0)
        super().__init__([g for g in groups if g["params"]], defaults)

    def _state(self, p, quantized):
        st = self.state[p]
        if not st:
            z = lambda dt: torch.zeros(p.shape, dtype=dt, device=p.device)
            st.update(m=z(torch.float32), v=z(torch.float32), updates=z(torch.int32))
            if quantized:
                rows, cols = p.shape
                u8 = lambda *s: torch.empty(s, dtype=torch.uint8, device=p.device)
                st.update(g_acc=z(torch.float32), acc_steps=z(torch.int32),
                          factor=torch.ones(p.shape, dtype=torch.int32, device=p.device),
                          w_prev=z(torch.float32), dist_w=z(torch.float32), dist_q=z(torch.float32),
                          codes_prev=u8(rows, cols // 2), scales_prev=u8(rows, cols // 32))
        return st

    def amplification_factors(self):
        """{parameter: N_w tensor in use} for the quantized weights (all ones before the first window closes)."""
        return {p: self.state[p]["factor"] for g in self.param_groups if g["quantized"] for p in g["params"] if self.state[p]}

    def load_state_dict(self, state_dict):
        """torch's loader converts every state tensor to its parameter's dtype; the integer arrays (update
        and step counts, factors, packed codes) are taken out before and put back unchanged after."""
        dropped = ("ones", "codes", "scales")              # arrays that earlier versions kept and nothing read
        slim = {"state": {k: {n: t for n, t in v.items() if n not in dropped} for k, v in state_dict["state"].items()},
                "param_groups": state_dict["param_groups"]}
        held = {k: {n: v.pop(n) for n in list(v) if torch.is_tensor(v[n]) and not v[n].is_floating_point()}
                for k, v in slim["state"].items()}
        super().load_state_dict(slim)
        params = [p for g in self.param_groups for p in g["params"]]
        for p in params:                                   # the kernels write in place: share nothing with the source
            for n, t in self.state[p].items():
                self.state[p][n] = t.clone()
        for k, tensors in held.items():
            for n, t in tensors.items():
                self.state[params[k]][n] = t.to(params[k].device).clone()

    @torch.no_grad()
    def step(self, closure=None):
        loss = None
        if closure is not None:
            with torch.enable_grad():
                loss = closure()
        for g in self.param_groups:
            phase = g["steps_done"] % g["t_update"]
            detecting = g["quantized"] and phase < g["t0"]
            (beta1, beta2), lr, eps, decay = g["betas"], g["lr"], g["eps"], g["weight_decay"]
            if not (lr >= 0 and 0 < beta1 < 1 and 0 < beta2 < 1 and eps >= 0 and decay >= 0):
                raise B.MxError("mx_ramping_adamw_step", B.MX_ERR_MODE)
            # one native call for the group: AdamW at the factors in use or, inside a window (whose first step also
            # sets the starting point w^0), AdamW at factor 1 with quantization and path lengths in the same pass.
            # A weight without a gradient stands still.
            params = g["params"] if detecting else [p for p in g["params"] if p.grad is not None]
            states = [self.state[p] or self._state(p, g["quantized"]) for p in params]
            B.host().ramping_step(params, states, 2 if detecting else int(g["quantized"]), phase == 0, g["scale_mode"],
                                  lr, beta1, beta2, eps, decay)
            if detecting and phase == g["t0"] - 1:
                for st in states:
                    B.mx_ramping_factor(st["dist_w"], st["dist_q"], g["k1"], g["k2"], g["n_max"], out=st["factor"])
            g["steps_done"] += 1
        return loss
