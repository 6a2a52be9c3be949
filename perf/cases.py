"""The work that programs ask of the Walsh-Hadamard output layer, as a list of measurable cases.

A case is one call (or one training step) of the layer at one token count, width and dtype:

    op = "forward"    y = alpha (.) (H x) + beta                              wht_affine_forward
         "residual"   y = resid + ...                                          wht_affine_forward_residual
         "stats"      (y, sum of squares of every row of y)                    wht_affine_forward_residual_stats
         "backward"   (dx, dalpha, dbeta)                                      wht_affine_backward
         "frozen"     dx alone: the parameters are not trained                 wht_affine_backward
         "params"     (dalpha, dbeta) alone: nothing below the layer is trained
         "step"       (y, dx, dalpha, dbeta): the forward and the backward call of one training step
         "train"      the same through autograd.WhtAffine and torch's autograd engine

Token counts and widths are those of the benchmark's workloads (synth.WORKLOADS), with odd counts
beside them: prompts and packed batches are rarely multiples of anything.
"""
import math

import torch

import paper_2603_08343_amd as wht
from paper_2603_08343_amd.autograd import WhtAffine

_DEV = "cuda:0"
_DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
_CHUNK = 1 << 25                        # elements of one block of the 64-bit reference
_POW2_BF16 = [1 << n for n in range(5, 15)]
_POW2_F32 = [1 << n for n in range(5, 14)]
_TWELVE = [768, 1536, 3072, 6144, 12288]
_LARGEST_BYTES = 2.0e9                  # no drawn case moves more than the largest listed one


def _case(name, op, N, d, dtype="bf16", outliers=False):
    return {"name": name, "op": op, "N": N, "d": d, "dtype": dtype, "outliers": outliers}


def listed():
    return [
        # the smallest configuration, float32: four heads of 64, one short sequence
        _case("tiny_f32_64x256", "forward", 64, 256, "f32"),
        # decoding, one sequence: the call an attention block makes for every token and layer, with
        # the residual add and the following norm's statistic fused in; latency is all there is
        _case("decode_1x4096", "stats", 1, 4096),
        # decoding, a batch of sequences at the Base width
        _case("decode_200x1536", "stats", 200, 1536),
        # one prompt of odd length, residual add fused in
        _case("prefill_3001x2048", "residual", 3001, 2048, outliers=True),
        # a batch of prompts (B=8 S=4096, 16 heads x 128), attention-like outliers
        _case("prefill_32768x2048", "forward", 32768, 2048, outliers=True),
        # fine-tuning on one packed sequence of odd length: a backward pass of ordinary size
        _case("finetune_4099x4096", "backward", 4099, 4096),
        # training steps of the small models: 16 heads x 64 and 12 heads x 64
        _case("step_32768x1024", "step", 32768, 1024),
        _case("step_32768x768", "step", 32768, 768),
        # a narrow model (4 heads x 64) on a ragged token batch
        _case("step_65537x256", "step", 65537, 256),
        # the wide layers: backward at 64 heads x 128, a whole step of the module at 48 heads x 128
        _case("backward_32768x8192", "backward", 32768, 8192),
        _case("train_32768x6144", "train", 32768, 6144),
        # float32 activations, 32 heads x 128
        _case("train_f32_16384x4096", "train", 16384, 4096, "f32"),
    ]


def draw(rng):
    """Any op, dtype and supported width; token counts spread over their logarithm from one token to
    what the largest listed case moves."""
    dtype = "f32" if rng.random() < 0.25 else "bf16"
    op = rng.choice(["forward", "residual", "stats", "backward", "frozen", "params", "step", "step", "train"])
    widths = _POW2_F32 if dtype == "f32" else _POW2_BF16 + _TWELVE
    d = rng.choice(widths)
    case = {"op": op, "N": 1, "d": d, "dtype": dtype, "outliers": rng.random() < 0.25}
    top = min(1 << 17, int(_LARGEST_BYTES / work(case)["bytes"]))
    case["N"] = max(1, min(top, int(round(math.exp(rng.uniform(0.0, math.log(top)))))))
    return case


# ------------------------------------------------------------------------------------------------
# inputs

def _inputs(case, seed):
    """x, dy, resid ~ N(0,1) (x with 1 % entries x 20 where the case says so), alpha ~ U(0.5, 1.5),
    beta ~ N(0, 0.02^2); tensors an op does not take are left out."""
    gen = torch.Generator(device=_DEV)
    gen.manual_seed(int(seed))
    N, d, op, dt = case["N"], case["d"], case["op"], _DTYPES[case["dtype"]]

    def normal():
        return torch.empty(N, d, dtype=dt, device=_DEV).normal_(generator=gen)

    s = {"alpha": torch.empty(d, device=_DEV).uniform_(0.5, 1.5, generator=gen),
         "beta": torch.empty(d, device=_DEV).normal_(0.0, 0.02, generator=gen)}
    if op != "frozen":
        s["x"] = normal()
        if case["outliers"]:
            # 1 % of the entries, a block of rows at a time: the mask's random numbers stay small
            for rows in s["x"].split(max(1, _CHUNK // d)):
                rows[torch.rand(rows.shape, device=_DEV, generator=gen) < 0.01] *= 20.0
    if op in ("backward", "frozen", "params", "step", "train"):
        s["dy"] = normal()
    if op in ("residual", "stats"):
        s["resid"] = normal()
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["op"] = case["op"]
    if case["op"] == "train":
        layer = WhtAffine(case["d"], device=_DEV)
        with torch.no_grad():
            layer.alpha.copy_(s["alpha"])
            layer.beta.copy_(s["beta"])
        s["layer"] = layer
        s["x"].requires_grad_(True)
    return s


def run(state):
    op = state["op"]
    if op == "forward":
        return wht.wht_affine_forward(state["x"], state["alpha"], state["beta"])
    if op == "residual":
        return wht.wht_affine_forward_residual(state["x"], state["alpha"], state["beta"], state["resid"])
    if op == "stats":
        return wht.wht_affine_forward_residual_stats(state["x"], state["alpha"], state["beta"], state["resid"])
    if op == "backward":
        return wht.wht_affine_backward(state["dy"], state["x"], state["alpha"])
    if op == "frozen":
        return wht.wht_affine_backward(state["dy"], None, state["alpha"], want_param_grads=False)[0]
    if op == "params":
        return wht.wht_affine_backward(state["dy"], state["x"], state["alpha"], want_dx=False)[1:]
    if op == "step":
        y = wht.wht_affine_forward(state["x"], state["alpha"], state["beta"])
        return (y, *wht.wht_affine_backward(state["dy"], state["x"], state["alpha"]))
    layer = state["layer"]
    y = layer(state["x"])
    grads = torch.autograd.grad(y, (state["x"], layer.alpha, layer.beta), state["dy"])
    return (y.detach(), *grads)


# ------------------------------------------------------------------------------------------------
# what a pass cannot do without

def work(case):
    """Each [N,d] tensor moved once (and the [d] and [N] vectors); d log2 d additions per transform."""
    N, d, op = case["N"], case["d"], case["op"]
    size = 4 if case["dtype"] == "f32" else 2
    streams, vectors, transforms = {
        "forward": (2, 2, 1), "residual": (3, 2, 1), "stats": (3, 2, 1), "backward": (3, 3, 2),
        "frozen": (2, 1, 1), "params": (2, 2, 1), "step": (5, 5, 3), "train": (5, 5, 3)}[op]
    nbytes = streams * N * d * size + vectors * d * 4 + (4 * N if op == "stats" else 0)
    stages = math.log2(d) if d % 3 else math.log2(d // 12) + 11
    return {"bytes": nbytes, "flops": transforms * N * d * stages + 2 * streams * N * d}


def tolerance(case):
    """bfloat16 results: one rounding of the output (2-norm 1.7e-3 of the result), four times that.
    float32 results: the roundings of the transform's log2 d additions and of the sums over the
    tokens (2-norm up to 1.7e-7 of the result observed), and between two orders of summation both
    sides' share: 1e-6."""
    return {"rel": 6.5e-3} if case["dtype"] == "bf16" else {"rel": 1e-6}


# ------------------------------------------------------------------------------------------------
# the same in 64 bits, from the definition

# the symmetric order-12 Hadamard matrix the layer documents for d = 12 * 2^m
_P12 = ("++++++++++++", "+--+-+-+-+-+", "+-+-++----++", "++--+--+-++-", "+-+++-++----", "+++---+--+-+",
        "+---+++-++--", "++-++---+--+", "+-----+++-++", "++-+-++---+-", "+-++----+++-", "+++--+-++---")


def _hadamard(z):
    """z <- H z along the last dimension, float64: pairwise sums and differences at strides 1, 2, 4, ...;
    for d = 12 * 2^m inside each of the 12 blocks, then the order-12 matrix across them."""
    n, d = z.shape
    blocks = 1 if d & (d - 1) == 0 else 12
    m = d // blocks
    h = 1
    while h < m:
        v = z.view(n, d // (2 * h), 2, h)
        z = torch.stack((v[:, :, 0] + v[:, :, 1], v[:, :, 0] - v[:, :, 1]), dim=2).view(n, d)
        h *= 2
    if blocks == 12:
        v = z.view(n, 12, m)
        rows = []
        for signs in _P12:
            acc = v[:, 0].clone()
            for k in range(1, 12):
                acc = acc + v[:, k] if signs[k] == "+" else acc - v[:, k]
            rows.append(acc)
        z = torch.stack(rows, dim=1).view(n, d)
    return z / math.sqrt(d)


def exact(case, seed):
    s = _inputs(case, seed)
    N, d, op = case["N"], case["d"], case["op"]
    alpha, beta = s["alpha"].double(), s["beta"].double()
    y = torch.empty(N, d, dtype=torch.float64, device=_DEV) if "x" in s and op not in ("backward", "params") else None
    sumsq = torch.empty(N, dtype=torch.float64, device=_DEV) if op == "stats" else None
    dx = torch.empty(N, d, dtype=torch.float64, device=_DEV) if op in ("backward", "frozen", "step", "train") else None
    dalpha = torch.zeros(d, dtype=torch.float64, device=_DEV)
    dbeta = torch.zeros(d, dtype=torch.float64, device=_DEV)
    step = max(1, _CHUNK // d)
    for lo in range(0, N, step):
        rows = slice(lo, min(N, lo + step))
        dy = s["dy"][rows].double() if "dy" in s else None
        if "x" in s:
            z = _hadamard(s["x"][rows].double())
            if y is not None:
                y[rows] = alpha * z + beta
                if "resid" in s:
                    y[rows] += s["resid"][rows].double()
                if sumsq is not None:
                    sumsq[rows] = (y[rows] ** 2).sum(dim=1)
            if dy is not None:
                dalpha += (dy * z).sum(dim=0)
                dbeta += dy.sum(dim=0)
        if dx is not None:
            dx[rows] = _hadamard(alpha * dy)
    if op in ("forward", "residual"):
        return y
    if op == "stats":
        return y, sumsq
    if op == "backward":
        return dx, dalpha, dbeta
    if op == "frozen":
        return dx
    if op == "params":
        return dalpha, dbeta
    return y, dx, dalpha, dbeta
