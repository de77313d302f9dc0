"""Helpers shared by the GPU parity tests: run one CLT train step through the
C ABI and through the CPU oracle on the same seeded inputs, and compare."""
from __future__ import annotations

import numpy as np
import torch

from oracle import clt_oracle as O
from workloads import clt_synth as S

MATS = ("W_enc", "W_dec")
MASK_BAND = 1e-3     # pre-activations this close to a decision boundary may fall either way


ELEM_RMS = 4.0       # weight of the local scale in the element-wise error bound (see max_elem)


def rel_l2(a, b):
    a = np.asarray(a, np.float64)
    b = np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30))


def max_elem(a, b):
    """Worst element of a against the reference b: max |a - b| / (|b| + ELEM_RMS * scale).

    A norm over a whole tensor lets one wrong element, or one wrong row of a large matrix, hide; this bounds
    every element on its own.  The size of an element's legitimate error is its own magnitude (rounding of the
    stored value) plus the magnitude of the terms that were summed into it and into the values it was computed
    from: an element near zero is a cancelled sum of terms that are not small.  That scale is taken from the
    reference: the RMS of the tensor (per layer / decoder block: the last two dimensions), or the RMS of the
    element's own row or column where that is larger -- tokens with heavy-tailed norms and outlier model
    dimensions make whole rows and columns of the step's matrices tens of times larger than the rest, and their
    rounding errors with them.  With bf16 operands (relative rounding 2^-9 each, a few such roundings per term)
    a sum carries an error of about 0.5 % of that scale, with a tail of five to six times that over millions of
    elements, hence the factor ELEM_RMS at the 2e-2 tolerance; a wrong element is off by about the scale itself.
    RMS values are taken over the reference's non-zero entries: the masked tensors of the step (z, dpre in the
    sparse regime) are exact zeros wherever the mask is off, and those zeros say nothing about the size of the
    terms behind the entries that are kept.  A reference that is identically zero must be reproduced exactly."""
    a = np.asarray(a, np.float64)
    b = np.asarray(b, np.float64)
    if b.size == 0:
        return 0.0
    if b.ndim < 2:
        a, b = a.reshape(1, -1), b.reshape(1, -1)
    sq, nzm = b * b, (b != 0)

    def rms(axis):
        n = nzm.sum(axis=axis, keepdims=True)
        return np.sqrt(sq.sum(axis=axis, keepdims=True) / np.maximum(n, 1))

    scale = np.maximum(rms((-2, -1)), np.maximum(rms(-1), rms(-2)))
    den = np.abs(b) + ELEM_RMS * scale
    err = np.abs(a - b)
    exact = den == 0.0
    if np.any(exact & (err != 0.0)):
        return float("inf")
    return float(np.max(np.where(exact, 0.0, err / np.where(exact, 1.0, den))))


def both_errs(errs, name, a, b):
    """Records the tensor-norm error and the worst-element error of a against b."""
    errs[name] = rel_l2(a, b)
    errs["elem:" + name] = max_elem(a, b)


def theta_for_density(x, W_enc, b_enc, rho):
    """Per-layer threshold (constant over features) at which a fraction `rho` of that layer's pre-activations
    lies above it: puts a test in the sparse regime of Sec. 3.2.  It only chooses an input (the threshold tensor
    handed to both sides), from a quantile of a subsample; neither side's result depends on how it was found."""
    L, F = x.shape[0], W_enc.shape[2]
    out = torch.empty((L, F), device=x.device, dtype=torch.float32)
    for l in range(L):
        s = (x[l] @ W_enc[l] + b_enc[l]).reshape(-1)
        if s.numel() > (1 << 22):
            s = s[:: s.numel() // (1 << 22)]
        kth = min(s.numel(), max(1, int(round(s.numel() * (1.0 - rho)))))
        out[l] = torch.kthvalue(s, kth).values
    return out


def fma_chain(a, b):
    """a [m, K] times b [K, n] in fp32 as one chain of fused multiply-adds per entry, in the order of K: acc = fma(a[:, k],
    b[k], acc).  The product of two fp32 numbers is exact in 64 bits; its sum with acc is rounded to odd there (the
    two-sum's error says whether and to which side it was inexact), so that rounding it to fp32 rounds once."""
    acc = np.zeros((a.shape[0], b.shape[1]), np.float32)
    for k in range(a.shape[1]):
        p, c = np.multiply.outer(a[:, k].astype(np.float64), b[k].astype(np.float64)), acc.astype(np.float64)
        s = p + c
        t = s - p
        err = (p - (s - t)) + (c - t)
        odd = (s.view(np.int64) & 1).astype(bool)
        s = np.where((err != 0) & ~odd, np.nextafter(s, np.where(err > 0, np.inf, -np.inf)), s)
        acc = s.astype(np.float32)
    return acc


def to_np(t):
    return t.detach().float().cpu().numpy().astype(np.float64)


GUARD_BYTES = 1024   # canary band on each side of every buffer the library writes
GUARD_BYTE = 0xA5


class GuardedBuffers:
    """Device buffers with a band of canary bytes directly before and after each one.  The library gets
    plain pointers and sizes, so a kernel that writes one element past a tensor (a ragged tile, a list
    one slot too long) would otherwise land in a neighbouring allocation unnoticed."""

    def __init__(self, dev):
        self.dev = dev
        self.items = []

    def empty(self, name, shape, dtype):
        n = int(np.prod(shape)) * torch.empty((), dtype=dtype).element_size()
        raw = torch.full((GUARD_BYTES + n + GUARD_BYTES,), GUARD_BYTE, dtype=torch.uint8, device=self.dev)
        self.items.append((name, raw, n))
        return raw[GUARD_BYTES:GUARD_BYTES + n].view(dtype).view(tuple(shape))

    def like(self, name, t, dtype=None):
        out = self.empty(name, t.shape, dtype or t.dtype)
        out.copy_(t)
        return out

    def check(self, after):
        torch.cuda.synchronize()
        for name, raw, n in self.items:
            ok = bool((raw[:GUARD_BYTES] == GUARD_BYTE).all()) and bool((raw[GUARD_BYTES + n:] == GUARD_BYTE).all())
            assert ok, f"canary bytes around '{name}' were overwritten by {after}"


class GpuRun:
    """One forward/loss/backward/Adam pass of the HIP library; results as numpy.  Every buffer the
    library may write (outputs, gradients, parameters and optimizer state, the workspace) sits between
    canary bands that are checked after each call."""

    def __init__(self, w: S.CLTWorkload, params, x, y, t=1, m=None, v=None, x_scale=None, y_scale=None,
                 theta=None, decode_mode=1, gather_density_threshold=0.004, fused=False, pre_steps=0,
                 reuse_decoder_norms=False, list_backward_density_threshold=0.0):
        """pre_steps: fused training steps run on the device before the step whose results are kept (that step
        then has step count t + pre_steps and starts from self.start_params / start_m / start_v)."""
        from paper_2603_21014_amd import binding as K
        dev = "cuda:0"
        T = torch.float32 if w.dtype == "f32" else torch.bfloat16
        TX = torch.int8 if w.int8_inputs else T
        gb = GuardedBuffers(dev)
        gp = {k: gb.like("params." + k, p, T if k in MATS else torch.float32) for k, p in params.items()}
        if theta is not None:
            gp["theta"].copy_(theta)
        state = lambda name, src: {k: (gb.empty(f"{name}.{k}", p.shape, torch.float32).zero_() if src is None
                                       else gb.like(f"{name}.{k}", src[k], torch.float32)) for k, p in gp.items()}
        gm, gv = state("m", m), state("v", v)
        master = None
        if w.master_weights:
            master = {k: gb.like("master." + k, params[k], torch.float32) for k in MATS}
        cfg = K.make_config(w.L, w.d, w.F, w.B, K.DTYPE_F32 if w.dtype == "f32" else K.DTYPE_BF16,
                            K.INPUT_INT8_ROWSCALE if w.int8_inputs else K.INPUT_NATIVE, w.master_weights, decode_mode,
                            gather_density_threshold, w.C, w.ste_eps, log_threshold=w.log_threshold, topk=w.topk or None,
                            reuse_decoder_norms=reuse_decoder_norms,
                            list_backward_density_threshold=list_backward_density_threshold)
        ws = gb.empty("workspace", (K.clt_workspace_bytes(cfg),), torch.uint8)
        step = K.CLTStep(w.L, w.d, w.F, w.B, dtype=w.dtype, int8_inputs=w.int8_inputs,
                         master_weights=w.master_weights, C_=w.C, ste_bandwidth=w.ste_eps, device=dev,
                         decode_mode=decode_mode, gather_density_threshold=gather_density_threshold,
                         log_threshold=w.log_threshold, topk=w.topk or None, workspace=ws,
                         reuse_decoder_norms=reuse_decoder_norms,
                         list_backward_density_threshold=list_backward_density_threshold)
        for name in ("z", "pre", "act_class", "y_hat", "l0", "loss_dev"):
            t_ = getattr(step, name)
            setattr(step, name, gb.empty(name, t_.shape, t_.dtype))
        step.grads = {k: gb.empty("grads." + k, g_.shape, g_.dtype) for k, g_ in step.grads.items()}
        xg, yg = x.to(dev, TX).contiguous(), y.to(dev, TX).contiguous()
        xs = x_scale.to(dev) if x_scale is not None else None
        ys = y_scale.to(dev) if y_scale is not None else None
        self.x_scale = to_np(xs) if xs is not None else None
        for i in range(pre_steps):
            step.train_step(xg, yg, gp, gm, gv, t + i, w.lr, w.lambda0, master, xs, ys, lambda1=w.lambda1)
            gb.check(f"training step {i + 1}")
        t += pre_steps
        cpu = lambda d_: {k: a.detach().float().cpu() for k, a in d_.items()}
        self.start_params, self.start_m, self.start_v = cpu(gp), cpu(gm), cpu(gv)
        K.clt_profile_enable(step.H, True)
        step.forward(xg, gp, xs)
        gb.check("clt_forward")
        self.loss = step.loss(yg, w.lambda0, ys, to_host=True, lambda1=w.lambda1, params=gp)
        gb.check("clt_loss")
        self.norms = to_np(K.clt_workspace_view(step.H, "norms"))
        self.d_yhat = to_np(K.clt_workspace_view(step.H, "d_yhat"))
        self.G = to_np(K.clt_workspace_view(step.H, "G"))
        if fused:     # backward and Adam in one call, Adam inside the weight-gradient GEMM epilogues
            step.backward_adam_step(xg, gp, gm, gv, t, w.lr, master, xs)
            gb.check("clt_backward_adam_step")
        else:
            step.backward(xg, gp, xs)
            gb.check("clt_backward")
        self.dpre = to_np(K.clt_workspace_view(step.H, "dpre"))
        torch.cuda.synchronize()
        self.pre, self.z, self.y_hat = to_np(step.pre), to_np(step.z), to_np(step.y_hat)
        cls = step.act_class.cpu().numpy()
        self.active, self.window = (cls & 1).astype(bool), (cls & 2).astype(bool)
        self.below = (cls & 4).astype(bool)
        self.l0 = step.l0.cpu().numpy()
        self.decode_switch = K.clt_workspace_view(step.H, "decode_switch").cpu().numpy()
        self.grads = {k: to_np(g) for k, g in step.grads.items()}
        if not fused:
            step.adam_step(t, w.lr, gp, gm, gv, master)
            gb.check("clt_adam_step")
        torch.cuda.synchronize()
        self.new_params = {k: to_np(p) for k, p in gp.items()}
        self.new_m = {k: to_np(a) for k, a in gm.items()}
        self.new_v = {k: to_np(a) for k, a in gv.items()}
        self.new_master = {k: to_np(a) for k, a in master.items()} if master else None
        self.kernel_launches = {k: n for k, (_, n) in K.clt_profile_query(step.H).items() if n}
        K.clt_profile_enable(step.H, False)
        self.step = step
        self.device_state = (gp, gm, gv, master)


class OracleRun:
    """The same step through oracle/clt_oracle.py.  If the GPU took the other valid
    decision for pre-activations inside MASK_BAND of a boundary, the oracle is
    asked to continue from that decision (it verifies the band itself)."""

    def __init__(self, w, params, x, y, t=1, m=None, v=None, gpu_active=None, gpu_window=None, theta=None,
                 x_np=None, y_np=None, gpu_below=None):
        npar = {k: to_np(p) for k, p in params.items()}
        if theta is not None:
            npar["theta"] = to_np(theta)
        xn = to_np(x) if x_np is None else x_np
        yn = to_np(y) if y_np is None else y_np
        self.x_np, self.y_np = xn, yn
        self.theta = O.threshold_value(npar["theta"], w.log_threshold)
        self.fwd = O.forward(xn, npar["W_enc"], npar["b_enc"], self.theta, npar["W_dec"], npar["b_dec"],
                             tie_break=gpu_active, band=MASK_BAND, topk=w.topk or None)
        self.n = O.decoder_norms(npar["W_dec"], w.L)
        tot, rec, sp = O.loss_terms(self.fwd["y_hat"], yn, self.fwd["z"], self.n, w.lambda0, w.C)
        dead = O.dead_feature_term(self.fwd["pre"], self.theta, self.n, w.lambda1)
        self.loss = (tot + dead, rec, sp, dead)
        self.bwd = O.backward(xn, yn, self.theta, npar["W_dec"], self.fwd, w.lambda0, w.C, w.ste_eps,
                              window_tie_break=None if w.topk else gpu_window, band=MASK_BAND, lambda1=w.lambda1,
                              log_threshold=w.log_threshold, below_tie_break=None if w.topk else gpu_below,
                              topk=bool(w.topk))
        zeros = {k: np.zeros_like(a) for k, a in npar.items()}
        m = zeros if m is None else {k: to_np(a) for k, a in m.items()}
        v = zeros if v is None else {k: to_np(a) for k, a in v.items()}
        self.new_params, self.new_m, self.new_v = {}, {}, {}
        for k in O.PARAM_NAMES:
            self.new_params[k], self.new_m[k], self.new_v[k] = O.adam_update(
                npar[k], self.bwd["d" + k], m[k], v[k], t, w.lr)
        self.params = npar


def compare_step(w, g: GpuRun, o: OracleRun, tol, check_adam=True):
    """Element-wise parity of every output of the step.  Returns the error table."""
    L = w.L
    theta = o.theta
    pre_o = o.fwd["pre"]
    errs = {}
    if w.topk:
        # the oracle has verified the selection against its own ranking outside the band around each row's
        # k-th value and that every row holds exactly k entries; there is no threshold, window or gradient of it
        assert (g.active == o.fwd["active"]).all() and (g.active.sum(axis=2) == w.topk).all()
        assert not g.window.any() and not g.below.any() and not g.grads["theta"].any()
        theta = np.full(theta.shape, np.inf)             # keeps the threshold-based checks below trivially true
        assert not o.bwd["window"].any()
    # masks: identical except inside the band around the boundary
    band = np.abs(pre_o - theta[:, None, :]) < MASK_BAND
    assert ((g.active == o.fwd["active"]) | band | bool(w.topk)).all(), "active mask differs outside the band"
    wband = np.abs(np.abs(pre_o - theta[:, None, :]) - 0.5 * w.ste_eps) < MASK_BAND
    assert ((g.window == o.bwd["window"]) | wband).all(), "window mask differs outside the band"
    assert ((g.below == (pre_o < theta[:, None, :])) | band | bool(w.topk)).all(), "below-threshold mask differs outside the band"
    assert not (g.below & g.active).any()
    assert (g.l0 == g.active.sum(axis=(1, 2))).all(), "l0_per_layer does not count the active mask"
    both_errs(errs, "pre", g.pre, pre_o)
    both_errs(errs, "z", g.z, o.fwd["z"])
    both_errs(errs, "norms", g.norms, o.n)
    for lp in range(L):
        both_errs(errs, f"y_hat[{lp}]", g.y_hat[lp], o.fwd["y_hat"][lp])
    for i, name in enumerate(("loss", "L_rec", "L_sp", "L_dead")):
        errs[name] = abs(g.loss[i] - o.loss[i]) / max(abs(o.loss[i]), 1e-30)
    both_errs(errs, "d_yhat", g.d_yhat, o.bwd["d_yhat"])
    # Column sums of the objective's decoder-norm derivative.  z sech^2(C z n) amplifies a relative
    # error of z by about 2 C z n, so with bf16 storage the reference is the oracle's sum over the
    # oracle's z rounded the way it is stored (the dead-feature part is linear and needs no such care).
    G_ref = o.bwd["G"]
    if w.dtype == "bf16":
        z_r = torch.from_numpy(o.fwd["z"]).to(torch.bfloat16).double().numpy()
        G_ref = G_ref - O.sparsity_norm_sums(o.fwd["z"], o.n, w.lambda0, w.C) \
            + O.sparsity_norm_sums(z_r, o.n, w.lambda0, w.C)
    both_errs(errs, "G", g.G, G_ref)
    # with int8 inputs the buffer holds dpre times the row scale of x (what dW_enc contracts with the codes)
    both_errs(errs, "dpre", g.dpre / g.x_scale[:, :, None] if w.int8_inputs else g.dpre, o.bwd["dpre"])
    for k in ("W_enc", "b_enc", "theta", "b_dec"):
        if k == "theta" and w.topk:
            continue                                     # exactly zero on both sides (asserted above)
        both_errs(errs, "d" + k, g.grads[k], o.bwd["d" + k])
    for p in range(O.num_blocks(L)):
        both_errs(errs, f"dW_dec[{p}]", g.grads["W_dec"][p], o.bwd["dW_dec"][p])
    bad = {k: e for k, e in errs.items() if not e <= tol}
    assert not bad, f"parity failures (tol {tol}): {bad}"
    if check_adam:
        check_adam_outputs(w, g, o, tol)
    return errs


def bf16_ulp(a):
    a = np.abs(np.asarray(a, np.float64))
    e = np.floor(np.log2(np.maximum(a, 2.0 ** -126)))
    return 2.0 ** (e - 7)


def check_adam_outputs(w, g: GpuRun, o: OracleRun, tol):
    """Moments within tol (they are linear / quadratic in the gradient).  The first
    update is -lr * g / (|g| + eps): it is compared where it is well conditioned
    (|g| >> eps and both gradients agree in sign and scale), up to the rounding of
    the stored parameter; everywhere it must stay within one learning rate."""
    for k in O.PARAM_NAMES:
        assert rel_l2(g.new_m[k], o.new_m[k]) <= tol, f"Adam m[{k}]"
        assert rel_l2(g.new_v[k], o.new_v[k]) <= 2 * tol, f"Adam v[{k}]"
        master = w.master_weights and k in MATS
        got = g.new_master[k] if master else g.new_params[k]
        want, old = o.new_params[k], o.params[k]
        g_o, g_g = o.bwd["d" + k], g.grads[k]
        cond = (np.abs(g_o) > 1e-5) & (np.abs(g_g - g_o) <= 0.5 * np.abs(g_o))
        if w.dtype == "bf16" and k in MATS and not master:
            quant = 0.51 * bf16_ulp(np.maximum(np.abs(got), np.abs(want)))
        else:
            quant = 2e-7 * np.abs(want) + 1e-12
        err = np.abs(got - want)
        assert (err[cond] <= quant[cond] + 2e-3 * w.lr).all(), f"Adam update {k}"
        assert (np.abs(got - old) <= 1.001 * w.lr + quant).all(), f"Adam step bound {k}"
        if master:
            rounded = g.new_params[k]
            assert (np.abs(rounded - got) <= 0.51 * bf16_ulp(got)).all(), f"bf16 copy of master {k}"


def run_both(w, theta=None, t=1, m=None, v=None, **gpu_kw):
    params = S.make_params(w)
    x, y = S.make_inputs(w)
    xs = ys = None
    xo = yo = None
    xin, yin = x, y
    if w.int8_inputs:
        xin, xs = S.quantize_rows_int8(x)
        yin, ys = S.quantize_rows_int8(y)
        xo = O.dequantize_rows(xin.numpy(), xs.numpy())
        yo = O.dequantize_rows(yin.numpy(), ys.numpy())
    g = GpuRun(w, params, xin, yin, t=t, m=m, v=v, x_scale=xs, y_scale=ys, theta=theta, **gpu_kw)
    o = OracleRun(w, params, x, y, t=t, m=m, v=v, gpu_active=g.active, gpu_window=g.window, theta=theta,
                  x_np=xo, y_np=yo, gpu_below=g.below)
    return g, o
