"""The work that users of this package have it do, as measurable cases.

A case is one pass of an FP8 linear layer (or of Calibrated Clipping) through
the package's public entry points, at the layer shapes of the 8B, 14B and 32B
models the repository's workloads name (hidden 4096 and 5120, FFN 12288,
17408 and 25600, query / key / value 4096 + 1024 + 1024), from a decode step
of a few sequences to a 16K-token training step.  Kinds:

  linear     Y = X W^T: quantize X, quantize W (fresh) or take W laid out
             once (a rollout's or an evaluation's weights), then the GEMM;
             scaling tensor, row, block (1x128 x 128x128) or pow2 (the same
             with power-of-two scales)
  splitk     a decode step's skinny product through gemm_splitk, with kept
             weights, outputs and workspace
  grouped    the fused query / key / value projections of one input
  quantized  the layer whose output is the next layer's FP8 operand
  train      one layer's training step: both layouts of X, W and W^T, the
             forward, both layouts of dY (E4M3 or E5M2), dgrad and wgrad
  clip       Calibrated Clipping over one batch of responses
"""
import math

import torch

import paper_2609_22870_amd as fp8q

T, ROW, B1, B128 = fp8q.TENSOR, fp8q.ROW, fp8q.BLOCK_1x128, fp8q.BLOCK_128x128
# (granularity of X, granularity of W, power-of-two scales)
SCALING = {"tensor": (T, T, False), "row": (ROW, ROW, False), "block": (B1, B128, False), "pow2": (B1, B128, True)}
E4M3_MAX, E5M2_MAX = 448.0, 57344.0
LAYERS = ((4096, 12288), (12288, 4096), (4096, 6144), (4096, 4096), (5120, 17408), (17408, 5120), (5120, 25600),
          (25600, 5120))
LARGEST = 3 * 2.0 * 16384 * 5120 * 25600  # flops of the largest listed case


def listed():
    return [
        # The smallest layer of the repository's workloads: latency, launches and host work.
        dict(name="tiny_tensor", kind="linear", scaling="tensor", fresh=True, M=128, K=256, N=256),
        # Rollout, a decode step of eight sequences: the fused projections.
        dict(name="decode8_qkv_grouped", kind="grouped", scaling="block", M=8, K=4096, N=4096, N2=1024, N3=1024),
        # Rollout, a decode step of 256 sequences: FFN up and down.
        dict(name="decode256_up", kind="linear", scaling="block", fresh=False, M=256, K=4096, N=12288),
        dict(name="decode256_down_splitk", kind="splitk", scaling="block", M=256, K=12288, N=4096),
        # Rollout prefill of a ragged number of tokens, the result handed on in FP8.
        dict(name="prefill_quantized_out", kind="quantized", M=3001, K=5120, N=17408),
        # Forward of one 16K-token sequence, weights quantized in the step (the headline workload).
        dict(name="forward_8b_up_block", kind="linear", scaling="block", fresh=True, M=16384, K=4096, N=12288),
        # The other scaling recipes, on other layers and token counts.
        dict(name="forward_8b_qkv_row", kind="linear", scaling="row", fresh=True, M=16384, K=4096, N=6144),
        dict(name="forward_8b_down_tensor", kind="linear", scaling="tensor", fresh=True, M=8192, K=12288, N=4096),
        dict(name="forward_14b_up_pow2", kind="linear", scaling="pow2", fresh=True, M=4096, K=5120, N=17408),
        # One layer's whole training step, 8B down-projection and 32B up-projection.
        dict(name="train_8b_down", kind="train", e5m2=False, M=8192, K=12288, N=4096),
        dict(name="train_32b_up_e5m2", kind="train", e5m2=True, M=16384, K=5120, N=25600),
        # Calibrated Clipping over one GRPO batch.
        dict(name="clip_grpo", kind="clip", prompts=256, group=8, min_len=512, max_len=8192),
    ]


def _log(rng, lo, hi, step):
    """A multiple of step, spread evenly over the logarithm of lo .. hi."""
    return max(step, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step)


def _layer(rng):
    """(K, N): a named layer, or any other width."""
    return rng.choice(LAYERS) if rng.random() < 0.6 else (_log(rng, 256, 16384, 128), _log(rng, 256, 16384, 128))


def draw(rng):
    case = _draw(rng)
    while any(case == {k: v for k, v in c.items() if k != "name"} for c in listed()):
        case = _draw(rng)
    return case


def _draw(rng):
    kind = rng.choice(("linear", "linear", "linear", "linear", "splitk", "grouped", "quantized", "train", "train", "clip"))
    K, N = _layer(rng)
    if kind == "linear":
        fresh = rng.random() < 0.6  # training and evaluation; else a rollout's decode or prefill
        M = _log(rng, 128, 16384, 1) if fresh else _log(rng, 1, 4096, 1)
        scaling = rng.choice(("block", "block", "row", "tensor", "pow2"))
        if scaling in ("row", "tensor") and rng.random() < 0.3:
            N += 16 * rng.randint(1, 7)  # widths that are no multiple of 128
        return dict(kind=kind, scaling=scaling, fresh=fresh, M=M, K=K, N=N)
    if kind == "splitk":
        return dict(kind=kind, scaling=rng.choice(("block", "block", "row")), M=_log(rng, 1, 512, 1), K=K, N=N)
    if kind == "grouped":
        kv = rng.choice((1024, 1024, 512, 256))
        return dict(kind=kind, scaling=rng.choice(("block", "block", "row")), M=_log(rng, 1, 16384, 1),
                    K=rng.choice((4096, 5120)),
                    N=rng.choice((4096, 5120, 8192)), N2=kv, N3=kv)
    if kind == "quantized":
        return dict(kind=kind, M=_log(rng, 16, 16384, 1), K=K, N=N)
    if kind == "train":
        M = _log(rng, 256, 16384, 128)
        M = min(M, int(LARGEST / (6.0 * K * N)) // 128 * 128)
        return dict(kind=kind, e5m2=rng.random() < 0.4, M=M, K=K, N=N)
    return dict(kind="clip", prompts=_log(rng, 8, 256, 1), group=8, min_len=_log(rng, 64, 512, 1),
                max_len=_log(rng, 1024, 8192, 1))


def _inputs(case, seed):
    """The tensors a layer's caller holds, from the seed alone: activations
    N(0, 1) with 1% of the channels fifty times as large, weights N(0, 0.02),
    output gradients N(0, 1e-3); for clip the per-token arrays of a batch."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def normal(rows, cols, sigma):
        return torch.randn((rows, cols), generator=g, device="cuda").mul_(sigma)

    if case["kind"] == "clip":
        n_resp = case["prompts"] * case["group"]
        lens = torch.randint(case["min_len"], case["max_len"] + 1, (n_resp,), generator=g, device="cuda")
        adv = torch.randn(n_resp, generator=g, device="cuda")
        adv[torch.rand(n_resp, generator=g, device="cuda") < 0.1] = 0.0
        adv = torch.repeat_interleave(adv, lens)
        a = [torch.randn(adv.numel(), generator=g, device="cuda") for _ in range(4)]
        r_bf16 = torch.exp(0.05 * a[1])
        return dict(adv=adv, w_tis=torch.clamp(torch.exp(0.02 * a[3]), max=2.0), pi=torch.sigmoid(3.0 + 2.0 * a[0]),
                    r_bf16=r_bf16, r_fp8=r_bf16 * torch.exp(0.03 * a[2]))
    M, K = case["M"], case["K"]
    x = normal(M, K, 1.0)
    hot = torch.randperm(K, generator=g, device="cuda")[: max(1, round(0.01 * K))]
    x[:, hot] *= 50.0
    t = dict(x=x.to(torch.bfloat16))
    for i, n in enumerate(_widths(case)):
        t["w%d" % i] = normal(n, K, 0.02).to(torch.bfloat16)
    if case["kind"] == "train":
        t["dy"] = normal(M, case["N"], 1e-3).to(torch.bfloat16)
    return t


def _widths(case):
    return [case[k] for k in ("N", "N2", "N3") if k in case]


def prepare(case, seed):
    t = _inputs(case, seed)
    kind = case["kind"]
    if kind == "clip":
        t["case"] = case
        t["workspace"] = torch.empty(fp8q.lib().fp8q_calibrate_clip_workspace(t["adv"].numel()), dtype=torch.uint8,
                                     device="cuda")
        return t
    s = dict(case=case, x=t["x"])
    if kind == "train":
        s.update(w=t["w0"], dy=t["dy"])
        return s
    if kind == "linear" and case["fresh"]:
        s["w"] = t["w0"]
        return s
    # a rollout's program: weights laid out once, buffers of a step kept
    gx, gw, pow2 = SCALING[case.get("scaling", "block")]
    M, K, N = case["M"], case["K"], case["N"]
    s["w"] = [fp8q.quantize(t["w%d" % i], gw, pow2=pow2) for i in range(len(_widths(case)))]
    s["xq"] = torch.empty((M, K), dtype=torch.uint8, device="cuda")
    s["sx"] = torch.empty(fp8q.scales_count(M, K, gx), dtype=torch.float32, device="cuda")
    if kind == "quantized":
        s["yq"] = torch.empty((M, N), dtype=torch.uint8, device="cuda")
        s["sy"] = torch.empty(fp8q.scales_count(M, N, B1), dtype=torch.float32, device="cuda")
    else:
        s["y"] = [torch.empty((M, n), dtype=torch.bfloat16, device="cuda") for n in _widths(case)]
    if kind == "splitk":
        s["workspace"] = torch.zeros(max(16, fp8q.gemm_splitk_workspace(M, N, K)), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "clip":
        return fp8q.calibrate_clip(s["adv"], s["w_tis"], s["pi"], s["r_bf16"], s["r_fp8"], 0.6, 1.8,
                                   workspace=s["workspace"])
    if kind == "train":
        return _train_step(s, case["e5m2"])
    gx, gw, pow2 = SCALING[case.get("scaling", "block")]
    gemm = fp8q.gemm_pow2 if pow2 else fp8q.gemm
    if kind == "linear" and case["fresh"]:
        xq, sx = fp8q.quantize(s["x"], gx, pow2=pow2)
        wq, sw = fp8q.quantize(s["w"], gw, pow2=pow2)
        return dict(y=gemm(xq, sx, gx, wq, sw, gw), xq=xq, sx=sx, wq=wq, sw=sw)
    xq, sx = fp8q.quantize(s["x"], gx, codes=s["xq"], scales=s["sx"], pow2=pow2)
    out = dict(xq=xq, sx=sx)
    wq, sw = s["w"][0]
    if kind == "linear":
        out["y"] = gemm(xq, sx, gx, wq, sw, gw, out=s["y"][0])
    elif kind == "splitk":
        out["y"] = fp8q.gemm_splitk(xq, sx, gx, wq, sw, gw, out=s["y"][0], workspace=s["workspace"])
    elif kind == "grouped":
        out["y"] = fp8q.gemm_grouped([(xq, sx, a, b) for a, b in s["w"]], gx, gw, outs=s["y"])
    else:
        out["yq"], out["sy"] = fp8q.gemm_quantized(xq, sx, gx, wq, sw, gw, codes=s["yq"], scales=s["sy"])
    return out


def _train_step(s, e5m2):
    xq, sx, xt, sxt = fp8q.quantize_dual(s["x"])
    wq, sw = fp8q.quantize(s["w"], B128)
    y = fp8q.gemm(xq, sx, B1, wq, sw, B128)
    wt, swt = fp8q.quantize(s["w"], B128, transposed=True)
    dq, sd, dt, sdt = fp8q.quantize_dual(s["dy"], e5m2=e5m2)
    if e5m2:
        dx = fp8q.gemm_formats(dq, sd, B1, wt, swt, B128, fp8q.A_E5M2)
        dw = fp8q.gemm_formats(dt, sdt, B1, xt, sxt, B1, fp8q.A_E5M2)
    else:
        dx = fp8q.gemm(dq, sd, B1, wt, swt, B128)
        dw = fp8q.gemm(dt, sdt, B1, xt, sxt, B1)
    return dict(y=y, dx=dx, dw=dw, xq=xq, sx=sx, xt=xt, sxt=sxt, wq=wq, sw=sw, wt=wt, swt=swt, dq=dq, sd=sd, dt=dt,
                sdt=sdt)


def _scales(rows, cols, g):
    return {T: 1, ROW: rows, B1: rows * cols // 128, B128: (rows // 128) * (cols // 128)}[g]


def work(case):
    """Inputs read once, outputs (codes and scales among them) written once."""
    kind = case["kind"]
    if kind == "clip":
        n = case["prompts"] * case["group"] * (case["min_len"] + case["max_len"]) / 2.0
        return {"bytes": 20.0 * n, "flops": 10.0 * n}
    M, K = case["M"], case["K"]
    gx, gw, _ = SCALING[case.get("scaling", "block")]
    if kind == "train":
        N = case["N"]
        b = 4.0 * M * K + 4.0 * N * K + 4.0 * M * N + 2.0 * (M * N + M * K + N * K)
        b += 4.0 * (2 * _scales(M, K, B1) + 2 * _scales(N, K, B128) + 2 * _scales(M, N, B1))
        return {"bytes": b, "flops": 6.0 * M * N * K}
    b = 3.0 * M * K + 4.0 * _scales(M, K, gx)
    for N in _widths(case):
        fresh = kind == "linear" and case["fresh"]
        b += (3.0 if fresh else 1.0) * N * K + 4.0 * _scales(N, K, gw)
        b += 1.0 * M * N + 4.0 * _scales(M, N, B1) if kind == "quantized" else 2.0 * M * N
    return {"bytes": b, "flops": 2.0 * M * K * sum(_widths(case))}


def tolerance(case):
    """Codes and scales are bytes and correctly rounded quotients: the same
    in any implementation.  GEMM outputs are bf16 (half an ulp is 2^-9, its
    2-norm 1.7e-3 off the exact product); another order of the fp32 sums
    moves some of them by an ulp."""
    if case["kind"] == "clip":
        return {"rel": 1e-12, "max": 1e-12}
    if case["kind"] == "quantized":
        return {"rel": 5e-3, "max": 2e-2, "differ": 1e-2}
    return {"rel": 5e-3, "max": 2e-2, "differ": 0.0}


def _units(v, g):
    """|v|'s maximum over each scaling unit, as v's shape broadcasts it."""
    a = v.abs()
    if g == T:
        return a.amax().reshape(1, 1)
    if g == ROW:
        return a.amax(dim=1, keepdim=True)
    r, c = a.shape
    if g == B1:
        return a.view(r, c // 128, 128).amax(dim=2).repeat_interleave(128, dim=1)
    return (a.view(r // 128, 128, c // 128, 128).amax(dim=(1, 3)).repeat_interleave(128, dim=0)
            .repeat_interleave(128, dim=1))


def _quantized(v, g, pow2=False, e5m2=False):
    """(v in 64 bits as its codes and scales give it back, its scale per
    element or unit): S = fp32(amax / F_max) or the power of two, 1 for a
    zero unit; the code the nearest FP8 value of fp32(v / S)."""
    f_max = E5M2_MAX if e5m2 else E4M3_MAX
    amax = _units(v, g).double()
    if pow2:
        m, e = torch.frexp(amax / f_max)
        s = torch.ldexp(torch.ones_like(m), torch.clamp(e - (m == 0.5).to(e.dtype), min=-127))
        s = torch.where(amax == 0, torch.ones_like(s), s)
    else:
        s = (amax / f_max).float().double()
        s = torch.where(s == 0, torch.ones_like(s), s)
    q = (v.double() / s).float().clamp(-f_max, f_max)
    q = q.to(torch.float8_e5m2 if e5m2 else torch.float8_e4m3fn)
    return q.double() * s, s


def _scale_vector(s, g):
    """The units' scales in the order the package lays them out."""
    if g == T:
        return s.reshape(1)
    if g == ROW:
        return s.reshape(-1)
    if g == B1:
        return s[:, ::128].t().reshape(-1)
    return s[::128, ::128].reshape(-1)


def _product(a, b):
    """a b^T in 64 bits, in strips of rows."""
    c = torch.empty((a.shape[0], b.shape[0]), dtype=torch.float64, device=a.device)
    for r in range(0, a.shape[0], 4096):
        torch.mm(a[r:r + 4096], b.t(), out=c[r:r + 4096])
    return c


def exact(case, seed):
    """run()'s floating outputs in 64 bits from plain torch (codes: None)."""
    t = _inputs(case, seed)
    kind = case["kind"]
    if kind == "clip":
        return _exact_clip(t)
    if kind == "train":
        return _exact_train(t, case["e5m2"])
    gx, gw, pow2 = SCALING[case.get("scaling", "block")]
    x, s = _quantized(t["x"], gx, pow2)
    sx = _scale_vector(s, gx)
    out = dict(xq=None, sx=sx)
    ys = []
    for i in range(len(_widths(case))):
        w, s = _quantized(t["w%d" % i], gw, pow2)
        ys.append(_product(x, w))
    if kind == "quantized":
        unit = _units(ys[0], B1) / E4M3_MAX
        return dict(out, yq=None, sy=_scale_vector(unit, B1))
    if kind == "linear" and case["fresh"]:
        out.update(wq=None, sw=_scale_vector(s, gw))
    return dict(out, y=ys if kind == "grouped" else ys[0])


def _exact_train(t, e5m2):
    out = dict(xq=None, xt=None, wq=None, wt=None, dq=None, dt=None)
    w, s = _quantized(t["w0"], B128)
    out.update(sw=_scale_vector(s, B128), swt=s[::128, ::128].t().reshape(-1))
    x, s = _quantized(t["x"], B1)
    out.update(y=_product(x, w), sx=_scale_vector(s, B1))
    d, s = _quantized(t["dy"], B1, e5m2=e5m2)
    out.update(dx=_product(d, w.t().contiguous()), sd=_scale_vector(s, B1))
    del x, w, d, s
    xt, s = _quantized(t["x"].t().contiguous(), B1)
    out["sxt"] = _scale_vector(s, B1)
    dt, s = _quantized(t["dy"].t().contiguous(), B1, e5m2=e5m2)
    out.update(dw=_product(dt, xt), sdt=_scale_vector(s, B1))
    return out


def _exact_clip(t):
    c = dict(c_low_ref=0.8, c_high_ref=1.24, l_min=0.5, l_max=0.9, h_min=1.2, h_max=2.0, step=0.02, delta_l=0.05,
             delta_h=0.1)
    a, rb, rf = t["adv"].double(), t["r_bf16"].double(), t["r_fp8"].double()
    wp = t["w_tis"].double() * t["pi"].double()
    neg, pos = a < 0, a > 0
    tb, tf = wp * rb * a, wp * rf * a

    def grid(lo, hi):
        return [lo + k * c["step"] for k in range(round((hi - lo) / c["step"]) + 1)]

    def smooth(b, best, delta):
        return b + min(max((best - b) / 2.0, -delta), delta)

    n_neg, n_pos = int(neg.sum()), int(pos.sum())
    ref = int((neg & (rb <= c["c_low_ref"])).sum())
    lower = grid(c["l_min"], c["l_max"])
    off = [abs(int((neg & (rf <= v)).sum()) - ref) for v in lower]
    l_star = lower[off.index(min(off))]
    rho_ref = float(tb[pos & (rb < c["c_high_ref"])].sum().abs() / tb[neg & (rb > c["c_low_ref"])].sum().abs())
    den = tf[neg & (rf > l_star)].sum().abs()
    upper = grid(c["h_min"], c["h_max"])
    rho = [float(tf[pos & (rf < v)].sum().abs() / den) for v in upper]
    off = [abs(v - rho_ref) for v in rho]
    kh = off.index(min(off))
    return dict(l_new=smooth(0.6, l_star, c["delta_l"]), h_new=smooth(1.8, upper[kh], c["delta_h"]), l_star=l_star,
                h_star=upper[kh], alpha_low=ref / n_neg, rho_bf16=rho_ref, rho_fp8=rho[kh], n_neg=n_neg, n_pos=n_pos,
                l_updated=1, h_updated=1)
