"""What a user of this library has it do, as cases that can be timed: convolution and FullyConnected layers run
through the calls of paper_1512_01274_amd.mxc, from one small fp32 layer to the 512-channel layers of a large network.

Three kinds of case:
  forward  one inference call, y = act(conv(x, w) + bias);
  train    what one training step asks of one layer: forward, bias gradient, weight gradient, input gradient.  With
           relu the layer stands inside a network: forward ends in a ReLU and the input gradient passes through the
           ReLU that produced x.  Layers of at most 4 channels (the network's input) bring x into its packed form
           once and hand it to forward and weight gradient;
  head     the last layer of a classifier for one step: FullyConnected, softmax, its gradient, bias, weight and input
           gradients, and the update of the fp32 weights and biases.
"""
import math

import torch

from paper_1512_01274_amd import mxc

LAYOUT = {"nchw": mxc.MXC_NCHW, "nhwc": mxc.MXC_NHWC}
DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}


def _conv(name, kind, dtype, layout, relu, N, C, H, W, K, R, stride, pad):
    return {"name": name, "kind": kind, "dtype": dtype, "layout": layout, "relu": relu, "N": N, "C": C, "H": H, "W": W, "K": K,
            "R": R, "stride": stride, "pad": pad}


def listed():
    return [
        # the single fp32 layer of the benchmark's first configuration: microseconds of work, launches and host time count
        _conv("single_f32", "train", "f32", "nhwc", False, 2, 16, 16, 16, 32, 3, 1, 1),
        # serving one image: a 13x13 layer of the AlexNet-style stack at batch 1
        _conv("serve_b1_3x3_384_256", "forward", "bf16", "nhwc", True, 1, 384, 13, 13, 256, 3, 1, 1),
        # fp32 training at batch 32 on NCHW tensors, the precision and batch of the paper's single-GPU comparison
        _conv("f32_nchw_3x3_192_384_b32", "train", "f32", "nchw", True, 32, 192, 13, 13, 384, 3, 1, 1),
        # first layers: strided 11x11 filter, and 3x3 at full resolution
        _conv("first_11x11s4_b128", "train", "bf16", "nhwc", False, 128, 3, 224, 224, 64, 11, 4, 2),
        _conv("first_3x3_b32", "train", "bf16", "nhwc", False, 32, 3, 224, 224, 64, 3, 1, 1),
        # the 5x5 layer of the AlexNet-style stack inside a network: bias, ReLU, masked input gradient
        _conv("5x5_64_192_b128", "train", "bf16", "nhwc", True, 128, 64, 27, 27, 192, 5, 1, 2),
        # the largest amount of matrix work: a 512-channel 3x3 layer of the VGG-style stack
        _conv("3x3_512_512_b64", "train", "bf16", "nhwc", True, 64, 512, 28, 28, 512, 3, 1, 1),
        # memory-bound 1x1 layers: inception reduction, bottleneck expansion, strided projection
        _conv("1x1_192_64_b128", "train", "bf16", "nhwc", True, 128, 192, 28, 28, 64, 1, 1, 0),
        _conv("1x1_64_256_b256", "train", "bf16", "nhwc", True, 256, 64, 56, 56, 256, 1, 1, 0),
        _conv("1x1s2_256_512_b256", "train", "bf16", "nhwc", False, 256, 256, 56, 56, 512, 1, 2, 0),
        # channel counts that are no multiple of 8, unequal image sides, floor remainder, NCHW tensors
        _conv("ragged_nchw_30_50_b64", "train", "bf16", "nchw", True, 64, 30, 45, 37, 50, 3, 2, 1),
        # the classifier's last layer with softmax and update
        {"name": "head_4096_1000_b128", "kind": "head", "N": 128, "C": 4096, "K": 1000},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, ragged):
    c = _log(rng, 16, 512)
    if ragged:
        return c
    step = 8 if c < 64 else 16 if c < 256 else 32
    return max(16, (c + step // 2) // step * step)


def _cost(case):
    """Work in units in which the largest listed case has about 1; fp32 and odd channel counts weigh more (they run far
    below the rates of bf16 on whole vectors)."""
    w = work(case)
    flops = w["flops"]
    if case["kind"] != "head":
        if case["dtype"] == "f32":
            flops *= 16
        elif (case["C"] > 4 and case["C"] % 8) or case["K"] % 8:
            flops *= 8
    return max(w["bytes"] / 3.0e9, flops / 5.3e11)


def draw(rng):
    what = rng.random()
    if what < 0.08:        # classifier heads
        case = {"kind": "head", "N": _log(rng, 8, 256), "C": _log(rng, 32, 512) * 16, "K": _log(rng, 10, 4096)}
        case["K"] = max(16, case["K"] // 8 * 8)
        return case
    case = {"kind": "train" if rng.random() < 0.7 else "forward", "dtype": "bf16", "layout": "nhwc", "relu": rng.random() < 0.6}
    N = _log(rng, 1, 256)
    if what < 0.2:         # first layers
        R, stride = rng.choice([(3, 1), (3, 2), (5, 1), (7, 2), (11, 4)])
        C, H, K = rng.choice([1, 3, 3, 3, 4]), _log(rng, 64, 224), 8 * rng.randint(2, 12)
        W = H if rng.random() < 0.6 else _log(rng, 64, 224)
        case.update(relu=False, pad=R // 2 if R < 11 else 2)
    else:
        R = rng.choice([1, 1, 1, 3, 3, 3, 3, 5])
        stride = 2 if R < 5 and rng.random() < 0.2 else 1
        ragged = rng.random() < 0.12
        C, K = _channels(rng, ragged), _channels(rng, ragged)
        H = _log(rng, 7, 80)
        W = H if rng.random() < 0.6 else _log(rng, 7, 80)
        case.update(pad=R // 2)
        if rng.random() < 0.2:
            case["dtype"] = "f32"
        if rng.random() < 0.25:
            case["layout"] = "nchw"
    case.update(N=N, C=C, H=H, W=W, K=K, R=R, stride=stride)
    while case["N"] > 1 and _cost(case) > 1.0:
        case["N"] //= 2
    return case


def _pq(c):
    return (c["H"] + 2 * c["pad"] - c["R"]) // c["stride"] + 1, (c["W"] + 2 * c["pad"] - c["R"]) // c["stride"] + 1


def _dims(c):
    return c["N"], c["C"], c["H"], c["W"], c["K"], c["R"], c["R"], c["stride"], c["pad"]


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape, sigma=1.0, dtype=torch.float32):
        return torch.randn(*shape, generator=g, device="cuda", dtype=dtype).mul_(sigma)

    if case["kind"] == "head":
        return _prepare_head(case, g, normal)
    N, C, H, W, K, R, _, stride, pad = dims = _dims(case)
    P, Q = _pq(case)
    dtype, layout = DTYPE[case["dtype"]], LAYOUT[case["layout"]]
    nhwc, train, first = layout == mxc.MXC_NHWC, case["kind"] == "train", C <= 4
    x = normal(*((N, H, W, C) if nhwc else (N, C, H, W)), dtype=dtype)
    if case["relu"]:
        x.relu_()          # inside a network x is a ReLU output
    s = {"case": case, "dims": dims, "dt": mxc.dtype_code(dtype), "lay": layout, "x": x, "relu": int(case["relu"]), "train": train,
         "first": first, "pq": (P, Q),
         "w": normal(*((K, R, R, C) if nhwc else (K, C, R, R)), sigma=math.sqrt(2.0 / (C * R * R)), dtype=dtype),
         "bias": normal(K, sigma=0.1),
         "y": torch.empty((N, P, Q, K) if nhwc else (N, K, P, Q), dtype=dtype, device="cuda")}
    size = lambda op: mxc.mxc_conv2d_workspace_bytes(op, *dims, s["dt"], layout)  # noqa: E731
    ops = [mxc.MXC_FWD]
    if train:
        s["dy"] = normal(*s["y"].shape, dtype=dtype)
        s["dx"] = torch.empty_like(x)
        s["dw"] = torch.empty(s["w"].shape, dtype=torch.float32, device="cuda")
        s["db"] = torch.empty(K, dtype=torch.float32, device="cuda")
        ops = [mxc.MXC_FWD, mxc.MXC_BWD_WEIGHT, mxc.MXC_BIAS_GRAD, mxc.MXC_BWD_DATA_RELU if case["relu"] else mxc.MXC_BWD_DATA]
        if first:
            ops[:2] = [mxc.MXC_FWD_PREPARED_INPUT, mxc.MXC_BWD_WEIGHT_PREPARED_INPUT]
            n = size(mxc.MXC_INPUT_PREPARED)
            s["xp"] = mxc.alloc_workspace(n) if n else x
            s["pack"] = n > 0
    s["ws"] = mxc.alloc_workspace(max(size(op) for op in ops))
    return s


def _prepare_head(case, g, normal):
    N, C, K = case["N"], case["C"], case["K"]
    bf = torch.bfloat16
    w = normal(K, C, sigma=math.sqrt(2.0 / C))
    s = {"case": case, "x": normal(N, C, dtype=bf).relu_(), "w": w, "wb": w.to(bf), "v": torch.zeros_like(w), "b": normal(K, sigma=0.1),
         "vb": torch.zeros(K, device="cuda"),
         "labels": torch.randint(0, K, (N,), generator=g, device="cuda", dtype=torch.int32),
         "dw": torch.empty_like(w), "db": torch.empty(K, device="cuda")}
    for name, cols in (("z", K), ("p", K), ("dz", K), ("dx", C)):
        s[name] = torch.empty(N, cols, dtype=bf, device="cuda")
    dims = (N, C, 1, 1, K, 1, 1, 1, 0, mxc.MXC_BF16, mxc.MXC_NHWC)
    s["ws"] = mxc.alloc_workspace(max(mxc.mxc_conv2d_workspace_bytes(op, *dims) for op in (
        mxc.MXC_FWD, mxc.MXC_BWD_DATA_RELU, mxc.MXC_BWD_WEIGHT, mxc.MXC_BIAS_GRAD)))
    return s


def run(s):
    if s["case"]["kind"] == "head":
        return _run_head(s)
    a = (*s["dims"], s["dt"], s["lay"])
    ws, first = s["ws"], s["first"] and s["train"]
    if first:
        if s["pack"]:
            mxc.mxc_conv2d_prepare_input(*a, s["x"], s["xp"])
        mxc.mxc_conv2d_fwd_prepared_input(*a, s["xp"], s["w"], s["bias"], s["relu"], s["y"], ws)
    else:
        mxc.mxc_conv2d_fwd_bias_act(*a, s["x"], s["w"], s["bias"], s["relu"], s["y"], ws)
    if not s["train"]:
        return s["y"]
    N, K, (P, Q) = s["dims"][0], s["dims"][4], s["pq"]
    mxc.mxc_bias_grad(N, K, P, Q, s["dt"], s["lay"], s["dy"], s["db"], ws)
    if first:
        mxc.mxc_conv2d_bwd_weight_prepared_input(*a, s["xp"], s["dy"], s["dw"], mxc.MXC_F32, ws)
    else:
        mxc.mxc_conv2d_bwd_weight(*a, s["x"], s["dy"], s["dw"], ws)
    if s["relu"]:
        mxc.mxc_conv2d_bwd_data_relu(*a, s["dy"], s["w"], s["x"], s["dx"], ws)
    else:
        mxc.mxc_conv2d_bwd_data(*a, s["dy"], s["w"], s["dx"], ws)
    return s["y"], s["db"], s["dw"], s["dx"]


def _run_head(s):
    N, C, K = s["case"]["N"], s["case"]["C"], s["case"]["K"]
    bf, ws = mxc.MXC_BF16, s["ws"]
    mxc.mxc_fc_fwd(N, C, K, bf, s["x"], s["wb"], s["b"], 0, s["z"], ws)
    mxc.mxc_softmax_fwd(N, K, bf, s["z"], s["p"])
    mxc.mxc_softmax_xent_bwd(N, K, bf, s["p"], s["labels"], 1.0 / N, s["dz"])
    mxc.mxc_bias_grad(N, K, 1, 1, bf, mxc.MXC_NHWC, s["dz"], s["db"], ws)
    mxc.mxc_fc_bwd_weight(N, C, K, bf, s["x"], s["dz"], s["dw"], ws)
    mxc.mxc_fc_bwd_data(N, C, K, bf, s["dz"], s["wb"], s["x"], s["dx"], ws)
    mxc.mxc_sgd_update(s["w"], s["dw"], s["v"], s["wb"], 0.05, 0.9, 1e-4)
    mxc.mxc_sgd_update(s["b"], s["db"], s["vb"], None, 0.05, 0.9, 0.0)
    return s["z"], s["p"], s["dz"], s["dx"], s["dw"], s["db"], s["w"], s["v"], s["wb"], s["b"]


def work(case):
    """Sums over the calls of one pass: each call reads its inputs and writes its outputs once."""
    if case["kind"] == "head":
        N, C, K = case["N"], case["C"], case["K"]
        fc = 2 * (N * C + K * C + N * K)
        return {"bytes": float(fc + 2 * N * K * 5 + fc + 2 * K * C + fc + 2 * N * C + 22 * K * C), "flops": 6.0 * N * C * K}
    N, C, H, W, K, R, _, stride, _ = _dims(case)
    P, Q = _pq(case)
    e = 4 if case["dtype"] == "f32" else 2
    x, w, y = N * C * H * W, K * C * R * R, N * K * P * Q
    if R == 1:
        touched = N * C * P * Q      # a strided 1x1 filter skips pixels
    else:
        touched = x
    flops = 2.0 * y * C * R * R
    n = e * (touched + w + y)
    if case["kind"] == "forward":
        return {"bytes": float(n), "flops": flops}
    n += e * y                                            # bias gradient
    n += e * (touched + y) + 4 * w                        # weight gradient
    n += e * (y + w + x) + (e * x if case["relu"] else 0)  # input gradient, and the mask it reads
    return {"bytes": float(n), "flops": 3.0 * flops}


def tolerance(case):
    if case["kind"] == "head":
        return {"rel": 1e-2, "max": 0.1}     # bf16 logits through a softmax: one rounding of a logit moves its probability
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 4e-3, "max": 2e-2}        # bf16 results: sums in another order round a value to its neighbour now and then
