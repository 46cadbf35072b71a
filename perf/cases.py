"""The timed cases of the library: matrix products with their epilogues, max reductions and
one-dimensional convolutions, called the way a program calls them (outputs and workspaces left to
the binding), over the sizes they are used at.

A case is a dict of plain values with an "op":

  "gemm"    C = act(A @ B + bias), optionally with the row sums of C; `bt`: the second factor is a
            linear layer's weight [N, K]; `splitk`: through the two-pass call
  "reduce"  maximum over one dimension of a dense tensor, values and first positions
  "conv"    one-dimensional convolution with bias and activation
"""
import math

import torch

from paper_2511_06345_amd import binding as pgk
from paper_2511_06345_amd.inputs import ACT_GELU_TANH, ACT_NONE, ACT_RELU, ACT_SILU

_ACTS = {"none": ACT_NONE, "relu": ACT_RELU, "gelu": ACT_GELU_TANH, "silu": ACT_SILU}
_TYPES = {"fp32": torch.float32, "bf16": torch.bfloat16}
_BYTES = {"fp32": 4, "bf16": 2}


def _gemm(dtype, M, N, K, batch=1, act="none", bias=True, rowsum=False, bt=False, splitk=False):
    return {"op": "gemm", "dtype": dtype, "M": M, "N": N, "K": K, "batch": batch, "act": act, "bias": bias,
            "rowsum": rowsum, "bt": bt, "splitk": splitk}


def _reduce(dtype, outer, red, inner):
    return {"op": "reduce", "dtype": dtype, "outer": outer, "red": red, "inner": inner}


def _conv(dtype, B, Cin, L, Cout, Kw, stride=1, pad=0, dilation=1, act="none"):
    return {"op": "conv", "dtype": dtype, "B": B, "Cin": Cin, "L": L, "Cout": Cout, "Kw": Kw, "stride": stride,
            "pad": pad, "dilation": dilation, "act": act}


def listed():
    cases = {
        # a small layer called on its own: the time is launches and latency
        "gemm_fp32_small": _gemm("fp32", 256, 256, 256, act="relu", rowsum=True),
        # a full-precision layer of a training or scientific program
        "gemm_fp32_square": _gemm("fp32", 4096, 4096, 4096, act="gelu"),
        # a large low-precision layer, the headline size of the benchmark
        "gemm_bf16_square": _gemm("bf16", 8192, 8192, 8192, act="silu"),
        # many rows onto few columns, with the row reduction in the epilogue
        "gemm_bf16_tall_rowsum": _gemm("bf16", 16384, 1024, 4096, act="relu", rowsum=True),
        # tiny outputs over a very long K (Gram matrices, weight gradients of a batch)
        "gemm_fp32_splitk": _gemm("fp32", 256, 256, 65536, batch=16, bias=False, rowsum=True, splitk=True),
        # one decoding step of a few sequences through a linear layer, weight as stored
        "gemm_bf16_decode": _gemm("bf16", 8, 11008, 4096, act="silu", bt=True),
        # projection onto a vocabulary of odd size
        "gemm_bf16_vocabulary": _gemm("bf16", 512, 50257, 768),
        # pooling over the middle dimension
        "reduce_fp32_strided": _reduce("fp32", 64, 4096, 1024),
        # the best entry of each row of vocabulary scores, rows of odd length
        "reduce_bf16_rows": _reduce("bf16", 2048, 50257, 1),
        # channel-heavy convolution, kernel 3 with "same" padding
        "conv_bf16_channels": _conv("bf16", 8, 512, 4096, 512, 3, pad=1, act="relu"),
        # long-sequence full-precision convolution with "same" padding
        "conv_fp32_long": _conv("fp32", 16, 64, 65536, 128, 3, pad=1, act="relu"),
        # first layer over a waveform: one input channel, strided
        "conv_fp32_waveform": _conv("fp32", 8, 1, 160000, 512, 10, stride=5, act="gelu"),
    }
    return [dict(case, name=name) for name, case in cases.items()]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """A size between lo and hi, spread over the logarithm: as drawn, or rounded to a multiple of 64."""
    n = _log(rng, lo, hi)
    return max(lo, min(hi, (n + 32) // 64 * 64)) if n >= 64 and rng.random() < 0.5 else n


# what a drawn case may cost: flops by type, and bytes
_MAX_FLOPS = {"fp32": 8e10, "bf16": 8e11}
_MAX_BYTES = 9e8


def _draw_gemm(rng):
    dtype = rng.choice(["fp32", "bf16"])
    kind = rng.choice(["layer", "layer", "decode", "batched", "longk"])
    if kind == "decode":
        M, N, K, batch = rng.randint(1, 32), _size(rng, 256, 32768), _size(rng, 256, 16384), 1
    elif kind == "batched":
        M, N, K, batch = _size(rng, 64, 2048), _size(rng, 64, 2048), _size(rng, 32, 2048), rng.randint(2, 64)
    elif kind == "longk":
        M, N, K, batch = _size(rng, 32, 512), _size(rng, 32, 512), _size(rng, 4096, 65536), rng.randint(1, 16)
    else:
        M, N, K, batch = _size(rng, 64, 16384), _size(rng, 64, 50257), _size(rng, 64, 8192), 1
    return _gemm(dtype, M, N, K, batch, act=rng.choice(list(_ACTS)), bias=rng.random() < 0.75,
                 rowsum=rng.random() < 0.4, bt=rng.random() < 0.5, splitk=kind == "longk" and rng.random() < 0.5)


def _draw_reduce(rng):
    dtype = rng.choice(["fp32", "bf16"])
    if rng.random() < 0.5:
        return _reduce(dtype, _size(rng, 1, 65536), _size(rng, 256, 1 << 22), 1)
    return _reduce(dtype, _size(rng, 1, 256), _size(rng, 16, 65536), _size(rng, 3, 4096))


def _draw_conv(rng):
    dtype = rng.choice(["fp32", "bf16"])
    Kw = rng.choice([1, 3, 3, 5, 7, 10])
    dilation = rng.choice([1, 1, 1, 2])
    Cin = rng.choice([1, 2, 3]) if rng.random() < 0.25 else _size(rng, 16, 512)
    stride = rng.choice([1, 1, 2, 5]) if Cin <= 3 else rng.choice([1, 1, 2])
    L = _size(rng, 512, 160000 if Cin <= 3 else 65536)
    return _conv(dtype, rng.randint(1, 16), Cin, L, _size(rng, 16, 512), Kw, stride=stride,
                 pad=rng.choice([0, dilation * (Kw - 1) // 2]), dilation=dilation, act=rng.choice(list(_ACTS)))


def draw(rng):
    while True:
        case = rng.choice([_draw_gemm, _draw_gemm, _draw_reduce, _draw_conv])(rng)
        cost = work(case)
        if cost["flops"] <= _MAX_FLOPS[case["dtype"]] and 1e5 <= cost["bytes"] <= _MAX_BYTES:
            return case


def _out_len(case):
    return (case["L"] + 2 * case["pad"] - case["dilation"] * (case["Kw"] - 1) - 1) // case["stride"] + 1


def work(case):
    e = _BYTES[case["dtype"]]
    if case["op"] == "gemm":
        M, N, K, batch = case["M"], case["N"], case["K"], case["batch"]
        nbytes = batch * (M * K + K * N + M * N) * e + (N * 4 if case["bias"] else 0)
        return {"bytes": nbytes + (batch * M * 4 if case["rowsum"] else 0), "flops": 2 * batch * M * N * K}
    if case["op"] == "reduce":
        outputs = case["outer"] * case["inner"]
        return {"bytes": outputs * (case["red"] * e + e + 4), "flops": outputs * case["red"]}
    x, w, y = case["B"] * case["Cin"] * case["L"], case["Cout"] * case["Cin"] * case["Kw"], case["B"] * case["Cout"] * _out_len(case)
    return {"bytes": (x + w + y) * e + case["Cout"] * 4, "flops": 2 * y * case["Cin"] * case["Kw"]}


def _inputs(case, seed):
    """The tensors of a case.  Activations and signals are uniform in [-1, 1), weights normal and
    scaled by the length of the sums they enter, biases normal with a tenth of that spread."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dtype = _TYPES[case["dtype"]]

    def uniform(*shape):
        return torch.empty(shape, dtype=torch.float32, device="cuda").uniform_(-1.0, 1.0, generator=gen).to(dtype)

    def normal(std, *shape):
        return torch.empty(shape, dtype=torch.float32, device="cuda").normal_(0.0, std, generator=gen)

    if case["op"] == "gemm":
        M, N, K, batch = case["M"], case["N"], case["K"], case["batch"]
        A = uniform(batch, M, K)
        B = normal(K ** -0.5, *((batch, N, K) if case["bt"] else (batch, K, N))).to(dtype)
        return A, B, normal(0.1, N) if case["bias"] else None
    if case["op"] == "reduce":
        return (uniform(case["outer"], case["red"], case["inner"]),)
    fan = case["Cin"] * case["Kw"]
    return (uniform(case["B"], case["Cin"], case["L"]),
            normal(fan ** -0.5, case["Cout"], case["Cin"], case["Kw"]).to(dtype), normal(0.1, case["Cout"]))


def prepare(case, seed):
    return {"case": case, "tensors": _inputs(case, seed)}


def run(state):
    case, tensors = state["case"], state["tensors"]
    if case["op"] == "gemm":
        A, B, bias = tensors
        call = ((pgk.gemm_splitk_bt if case["bt"] else pgk.gemm_splitk) if case["splitk"]
                else (pgk.gemm_fused_bt if case["bt"] else pgk.gemm_fused))
        C, rowsum = call(A, B, bias, _ACTS[case["act"]], rowsum=case["rowsum"])
        return (C, rowsum) if case["rowsum"] else (C,)
    if case["op"] == "reduce":
        return pgk.reduce_max(tensors[0], 1)
    x, w, bias = tensors
    return (pgk.conv1d(x, w, bias, _ACTS[case["act"]], case["stride"], case["pad"], case["dilation"]),)


# Measured on the listed and some drawn cases as the distance from `exact`, times about four.
# fp32: the products' sums; bf16: the rounding of the stored output (half a unit in the last
# place of 8 bits is 2^-9), as the sums are kept in 32 bits.
_TOLERANCE = {"fp32": {"rel": 7e-6, "max": 7e-5}, "bf16": {"rel": 7e-3, "max": 1.6e-2}}


def tolerance(case):
    return "exact" if case["op"] == "reduce" else _TOLERANCE[case["dtype"]]


def _act64(x, act):
    if act == "relu":
        return x.clamp_min_(0.0)
    if act == "gelu":
        return torch.nn.functional.gelu(x, approximate="tanh")
    return torch.nn.functional.silu(x) if act == "silu" else x


def exact(case, seed):
    tensors = _inputs(case, seed)
    if case["op"] == "gemm":
        A, B, bias = tensors
        C = torch.empty((case["batch"], case["M"], case["N"]), dtype=torch.float64, device=A.device)
        for b in range(case["batch"]):
            x = A[b].double() @ (B[b].double().t() if case["bt"] else B[b].double())
            C[b] = _act64(x + bias.double() if case["bias"] else x, case["act"])
        return (C, C.sum(-1)) if case["rowsum"] else (C,)
    if case["op"] == "reduce":
        X = tensors[0]
        best = X.amax(1)
        first = torch.empty(best.shape, dtype=torch.int64, device=X.device)
        place = torch.arange(case["red"], device=X.device).view(-1, 1)
        for o in range(case["outer"]):
            first[o] = torch.where(X[o] == best[o], place, case["red"]).amin(0)
        return best.double(), first
    x, w, bias = tensors
    stride, dilation, pad = case["stride"], case["dilation"], case["pad"]
    span = (_out_len(case) - 1) * stride + 1
    xp, w = torch.nn.functional.pad(x, (pad, pad)), w.double()
    y = torch.empty((case["B"], case["Cout"], _out_len(case)), dtype=torch.float64, device=x.device)
    for b in range(case["B"]):
        row = bias.double().view(-1, 1).expand(-1, y.shape[2])
        for k in range(case["Kw"]):
            row = row + w[:, :, k] @ xp[b, :, k * dilation:k * dilation + span:stride].double()
        y[b] = _act64(row, case["act"])
    return (y,)
