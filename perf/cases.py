"""The work that is timed: forward passes of the library's layers as a program asks for them.

A program meets the library in one of these forms, and every case is one of them:

  calls   the four calls of the method one after the other (pack, K, alpha, convolution), outputs and
          workspace allocated by the binding: a first try, a single layer, a test harness
  step    input and filters both new: one prepare call, then the convolution on expanded filters
          (bench.py's step)
  infer   the filters prepared once and kept, a new input per pass: inference on one layer
  chain   a stack of layers that hand packed signs to each other, filters kept, fp32 in and out
  image   a whole forward pass on an image of few channels (first layers, the paper's own workload)
  bwn     a Binary-Weight-Network layer: fp32 input, sign filters kept
  fp32    the real-valued convolution that the binary one is compared with

Sizes are those of paper_2007_14178_amd/workloads.py and bench.py, and generic ones where these have
none (odd sides, channel and filter counts that are no multiple of 32).
"""
import math

import torch

from paper_2007_14178_amd import binding as xb


def _case(name, form, N, C, H, W, F, k, stride=1, pad=None, k_in_conv=False, want_dot=False, layers=1):
    case = {"form": form, "N": N, "C": C, "H": H, "W": W, "F": F, "k": k, "stride": stride,
            "pad": k // 2 if pad is None else pad, "k_in_conv": k_in_conv, "want_dot": want_dot, "layers": layers}
    return {"name": name, **case} if name else case


def listed():
    return [
        # one small layer, one image, by the four calls: latency, launches and the host's share
        _case("calls_32", "calls", 1, 64, 32, 32, 64, 3),
        # a ragged layer (nothing a multiple of 32) by the four calls, with the binary dot products
        _case("calls_ragged", "calls", 5, 100, 37, 53, 75, 3, want_dot=True),
        # the wide-kernel layer of the kernel-size sweep with new filters on every pass
        _case("step_56_k5", "step", 16, 128, 56, 56, 128, 5, k_in_conv=True),
        # a ResNet-18-shaped stride-2 layer at inference
        _case("infer_28_s2", "infer", 64, 128, 28, 28, 256, 3, stride=2, k_in_conv=True),
        # an AlexNet-shaped layer at inference: odd 13 x 13 planes
        _case("infer_13", "infer", 128, 384, 13, 13, 384, 3, k_in_conv=True),
        # the large-channel benchmark layer, everything in the step
        _case("step_28_large", "step", 128, 512, 28, 28, 512, 3),
        # three ResNet-18-shaped layers that pass packed signs on
        _case("chain_14", "chain", 64, 256, 14, 14, 256, 3, k_in_conv=True, layers=3),
        # the paper's own workload at its largest size
        _case("image_2048", "image", 1, 1, 2048, 2048, 1, 3),
        # a first layer on colour images of odd size, 7 x 7 filters, stride 2
        _case("image_rgb", "image", 16, 3, 227, 227, 64, 7, stride=2),
        # an AlexNet-shaped layer with real-valued input
        _case("bwn_13", "bwn", 128, 384, 13, 13, 384, 3),
        # the float comparison on the sweep's wide-kernel layer and on the large-channel layer
        _case("fp32_56_k5", "fp32", 16, 128, 56, 56, 128, 5),
        _case("fp32_28_large", "fp32", 128, 512, 28, 28, 512, 3),
    ]


def _log(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


#: most multiply-accumulates and most output values of a drawn case, by form
_MOST = {"calls": (60e9, 30e6), "step": (200e9, 50e6), "infer": (200e9, 50e6), "chain": (120e9, 50e6),
         "image": (4e9, 60e6), "bwn": (100e9, 50e6), "fp32": (12e9, 30e6)}


def draw(rng):
    form = rng.choice(["calls", "step", "infer", "infer", "chain", "image", "bwn", "fp32"])
    if form == "image":
        C, k = rng.choice([1, 1, 3, 3, 2, 4]), rng.choice([3, 3, 5, 7])
        N = 1 if C == 1 else _log(rng, 1, 32)
        H = _log(rng, 200, 2048) if C == 1 else _log(rng, 64, 512)
        W = max(32, int(H * rng.uniform(0.7, 1.4)))
        F = rng.choice([1, 1, 2, 4]) if C == 1 else _log(rng, 8, 96)
        stride = 1 if C == 1 else rng.choice([1, 2, 2, 4])
    else:
        k = rng.choice([3, 3, 3, 5, 7, 1])
        N, C, F = _log(rng, 1, 128), _log(rng, 32, 512), _log(rng, 32, 512)
        if rng.random() < 0.6:      # most layers have channel counts that are multiples of 32
            C, F = max(32, C // 32 * 32), max(32, F // 32 * 32)
        H = _log(rng, 7, 64)
        W = H if rng.random() < 0.6 else max(7, int(H * rng.uniform(0.7, 1.4)))
        stride = rng.choice([1, 1, 1, 2])
        if form == "chain":
            k, stride, F = rng.choice([3, 3, 5, 1]), 1, C
    case = _case(None, form, N, C, H, W, F, k, stride, pad=rng.choice([k // 2, k // 2, k // 2, 0]) if form != "chain" else k // 2,
                 k_in_conv=rng.random() < 0.5, want_dot=form in ("calls", "image") and rng.random() < 0.3,
                 layers=rng.choice([2, 3]) if form == "chain" else 1)
    macs, outs = _MOST[form]
    while _macs(case) > macs or _outs(case) > outs:
        if case["N"] > 1:
            case["N"] = max(1, case["N"] * 2 // 3)
        else:
            case["F"] = max(1, case["F"] // 2)
            if form == "chain":
                case["C"] = case["F"]
    return case


def _shape(c):
    return xb.Shape(c["N"], c["C"], c["H"], c["W"], c["F"], c["k"], c["k"], c["stride"], c["stride"], c["pad"], c["pad"])


def _out_dims(c):
    return (c["H"] + 2 * c["pad"] - c["k"]) // c["stride"] + 1, (c["W"] + 2 * c["pad"] - c["k"]) // c["stride"] + 1


def _outs(c):
    OH, OW = _out_dims(c)
    return c["N"] * c["F"] * OH * OW


def _macs(c):
    return c["layers"] * _outs(c) * c["C"] * c["k"] * c["k"]


def _tensors(c, seed):
    """The fp32 input (5 % exact zeros, as benchmark layer 5 has them) and the filters of every layer."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    I = torch.randn((c["N"], c["C"], c["H"], c["W"]), generator=g, device="cuda")
    I.masked_fill_(torch.rand(I.shape, generator=g, device="cuda") < 0.05, 0.0)
    return I, [torch.randn((c["F"], c["C"], c["k"], c["k"]), generator=g, device="cuda") * 0.05 for _ in range(c["layers"])]


def prepare(case, seed):
    c, s = case, _shape(case)
    I, Wts = _tensors(c, seed)
    OH, OW = _out_dims(c)

    def f32(*dims):
        return torch.empty(dims, dtype=torch.float32, device="cuda")

    def i32(*dims):
        return torch.empty(dims, dtype=torch.int32, device="cuda")

    st = {"case": c, "s": s, "I": I, "Wts": Wts}
    if c["form"] == "calls":
        return st
    st["out"] = f32(c["N"], c["F"], OH, OW)
    if c["form"] == "fp32":
        return st
    if c["form"] == "image":
        st["dot"] = i32(c["N"], c["F"], OH, OW) if c["want_dot"] else None
    if c["form"] in ("image", "bwn"):
        st["Wpk"], st["alpha"], _ = xb.xnor_filter_prepare(Wts[0])
        return st
    # buffers that the layers of a program share
    st["Ipk"], st["A"] = i32(c["N"], c["H"], c["W"], s.Cw), f32(c["N"], c["H"], c["W"])
    st["K"] = f32(c["N"], OH, OW)
    chain = c["form"] == "chain"
    # not every shape has a kernel that works on expanded filters; those go by the packed ones
    nbytes = xb.xnor_conv2d_workspace_bytes(s)
    if chain and nbytes:
        nbytes = xb.xnor_conv2d_chain_workspace_bytes(s)
    st["workspaces"] = [torch.empty((nbytes,), dtype=torch.uint8, device="cuda") if nbytes else None for _ in Wts]
    if c["form"] == "step":
        st["Wpk"], st["M"], st["alpha"] = i32(c["F"], c["k"], c["k"], s.Cw), f32(c["F"], c["k"], c["k"]), f32(c["F"])
        return st
    st["Wpks"], st["alphas"] = [], []
    for Wt, ws in zip(Wts, st["workspaces"]):
        Wpk, alpha, _ = xb.xnor_filter_prepare(Wt)
        if ws is not None:
            xb.xnor_filter_expand(Wpk, s, ws)
        st["Wpks"].append(Wpk)
        st["alphas"].append(alpha)
    if chain:
        st["packed"] = [i32(c["N"], OH, OW, s.Cw) for _ in range(2)]
        st["means"] = [f32(c["N"], OH, OW) for _ in range(2)]
    return st


def run(st):
    c, s, I, Wt = st["case"], st["s"], st["I"], st["Wts"][0]
    form = c["form"]
    if form == "calls":
        Ipk, Wpk = xb.xnor_binarize_pack(I), xb.xnor_binarize_pack(Wt)
        K, A = xb.xnor_scale_K(I, s)
        alpha = xb.xnor_alpha(Wt)
        out, dot = xb.xnor_conv2d_fwd(Ipk, Wpk, K, alpha, s, want_dot=c["want_dot"])
        return {"out": out, "dot": dot, "K": K, "A": A, "alpha": alpha, "Ipk": Ipk, "Wpk": Wpk}
    if form == "image":
        out, dot = xb.xnor_forward_image(I, st["Wpk"], st["alpha"], s, st["out"], st["dot"])
        return {"out": out, "dot": dot}
    if form == "bwn":
        return {"out": xb.xnor_bwn_conv2d_fwd(I, st["Wpk"], st["alpha"], s, st["out"])}
    if form == "fp32":
        return {"out": xb.xnor_conv2d_fp32_fwd(I, Wt, s, st["out"])}
    ws = st["workspaces"][0]
    k_in_conv = c["k_in_conv"] and ws is not None
    K = None if k_in_conv else st["K"]
    if form == "step":
        _, _, A, Wpk, alpha, _ = xb.xnor_prepare(I, Wt, s, st["Ipk"], st["A"], K, st["Wpk"], st["M"], st["alpha"],
                                                 want_K=not k_in_conv, workspace=ws)
    else:
        _, _, A = xb.xnor_input_prepare(I, s, st["Ipk"], st["A"], K, want_K=not k_in_conv)
        Wpk, alpha = st["Wpks"][0], st["alphas"][0]
    if form != "chain":
        if ws is None:
            out, _ = xb.xnor_conv2d_fwd(st["Ipk"], Wpk, st["K"], alpha, s, st["out"], workspace=None)
        else:
            out, _ = xb.xnor_conv2d_fwd_expanded(st["Ipk"], ws, K, alpha, s, st["out"], A=A if k_in_conv else None)
        return {"out": out, "A": A, "alpha": alpha}
    packed, last = st["Ipk"], c["layers"] - 1
    for i in range(last):
        to, mean = st["packed"][i % 2], st["means"][i % 2]
        if i and not k_in_conv:
            xb.xnor_box_filter_K(A, s, K)
        if ws is not None:
            xb.xnor_conv2d_fwd_chain(packed, None, K, st["alphas"][i], s, to, mean, st["workspaces"][i], A if k_in_conv else None)
        else:       # no chained kernel for the shape: the fp32 output goes through the input pass
            out, _ = xb.xnor_conv2d_fwd(packed, st["Wpks"][i], K, st["alphas"][i], s, st["out"], workspace=None)
            xb.xnor_input_prepare(out, s, to, mean, K)
        packed, A = to, mean
    if ws is None:
        out, _ = xb.xnor_conv2d_fwd(packed, st["Wpks"][last], K, st["alphas"][last], s, st["out"], workspace=None)
    else:
        if not k_in_conv:
            xb.xnor_box_filter_K(A, s, K)
        out, _ = xb.xnor_conv2d_fwd_expanded(packed, st["workspaces"][last], K, st["alphas"][last], s, st["out"],
                                             A=A if k_in_conv else None)
    return {"out": out, "packed": packed, "A": A}


def work(case):
    c = case
    OH, OW = _out_dims(c)
    pixels, weights = c["N"] * c["H"] * c["W"], c["F"] * c["C"] * c["k"] ** 2
    moved = 4 * pixels * c["C"] + 4 * _outs(c) * (2 if c["want_dot"] else 1)
    if c["form"] in ("calls", "step", "fp32"):
        moved += 4 * weights                                    # fp32 filters
    else:
        moved += c["layers"] * (weights // 8 + 4 * c["F"])      # sign bits and alpha
    if c["form"] in ("calls", "step", "infer", "chain"):
        moved += 4 * pixels                                     # the channel mean, which is returned
    if c["form"] in ("calls", "chain"):
        moved += c["N"] * c["H"] * c["W"] * ((c["C"] + 31) // 32) * 4
    if c["form"] == "calls":
        moved += 4 * c["N"] * OH * OW + weights // 8 + 4 * c["F"]
    return {"bytes": float(moved), "flops": 2.0 * _macs(c)}


def tolerance(case):
    if case["form"] in ("bwn", "fp32"):
        # signed sums of up to some thousand fp32 terms: the rounding of the sum, not of its terms
        # (5e-7 to 1.2e-6 off the 64-bit result)
        return {"rel": 5e-6, "max": 1e-4}
    # sums of magnitudes and a product of three fp32 factors (up to 7.4e-8 off); whole numbers stay the same
    return {"rel": 4e-7, "max": 4e-6}


def _conv64(x, w, c):
    """x [N][C][H][W], w [F][C][k][k] in 64 bits: the zero-padded convolution, tap by tap."""
    OH, OW = _out_dims(c)
    p, st, k = c["pad"], c["stride"], c["k"]
    xp = torch.nn.functional.pad(x, (p, p, p, p)).permute(1, 0, 2, 3)
    acc = torch.zeros((w.shape[0], x.shape[0] * OH * OW), dtype=torch.float64, device=x.device)
    for ky in range(k):
        for kx in range(k):
            tap = xp[:, :, ky:ky + st * (OH - 1) + 1:st, kx:kx + st * (OW - 1) + 1:st].reshape(x.shape[1], -1)
            acc += w[:, :, ky, kx].contiguous() @ tap.contiguous()
    return acc.reshape(w.shape[0], x.shape[0], OH, OW).permute(1, 0, 2, 3)


def _sign64(x):
    return torch.where(x >= 0, 1.0, -1.0).to(torch.float64)


def _box64(A, c):
    return _conv64(A[:, None], torch.full((1, 1, c["k"], c["k"]), 1.0 / c["k"] ** 2, dtype=torch.float64, device=A.device), c)


def exact(case, seed):
    c = case
    I, Wts = _tensors(c, seed)
    if c["form"] == "fp32":
        return {"out": _conv64(I.double(), Wts[0].double(), c)}
    alphas = [w.double().abs().mean(dim=(1, 2, 3)) for w in Wts]
    signs = [_sign64(w) for w in Wts]
    if c["form"] == "bwn":
        return {"out": _conv64(I.double(), signs[0], c) * alphas[0][None, :, None, None]}
    A, x = I.double().abs().mean(dim=1), _sign64(I)
    for i in range(c["layers"]):
        K, A_in = _box64(A, c), A
        out = _conv64(x, signs[i], c) * K * alphas[i][None, :, None, None]
        A, x = out.abs().mean(dim=1), _sign64(out)
    if c["form"] == "calls":
        return {"out": out, "dot": None, "K": K[:, 0], "A": A_in, "alpha": alphas[0], "Ipk": None, "Wpk": None}
    if c["form"] == "image":
        return {"out": out, "dot": None}
    if c["form"] == "chain":
        return {"out": out, "packed": None, "A": A_in}
    return {"out": out, "A": A_in, "alpha": alphas[0]}
