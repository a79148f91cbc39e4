"""The calls whose speed is watched: layout chains run as one gather, and products that read and store through
composed maps, each through the package's public entry points, from one small image batch to a few hundred
megabytes.  `listed` names them, `draw` gives more of the same ranges, `prepare` makes what a program holds
before the call (inputs on the GPU, composed maps, output buffers) and `run` is the call itself."""
from __future__ import annotations

import torch

from paper_2002_12798_amd import binding as B
from paper_2002_12798_amd import device

DTYPES = {"fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}


def listed():
    return [
        # The smallest call: a few hundred kilobytes of activations flattened to a token sequence, cropped and
        # padded in the channel (launch latency and the way to the launch are what it costs).
        dict(name="tokens_small", kind="tokens", dtype="fp32", batch=8, channels=16, size=32, pad=4),
        # A channel-major activation made channels-last with the zero border of the 3 x 3 convolution after it.
        dict(name="nhwc_pad", kind="nhwc_pad", dtype="bf16", batch=32, channels=256, size=56, pad=1),
        # The same in fp32 at training batch: the largest transfer.
        dict(name="nhwc_pad_large", kind="nhwc_pad", dtype="fp32", batch=128, channels=256, size=56, pad=1),
        # Q, K and V of a projection split by heads into three tensors of their own, one call.
        dict(name="qkv_split", kind="qkv_split", dtype="bf16", batch=16, seq=512, heads=12, dim=64),
        # The way back: the heads of an attention output merged into rows.
        dict(name="head_merge", kind="head_merge", dtype="bf16", batch=16, seq=512, heads=12, dim=64),
        # The branches of an inception block joined along the channels and made channels-last.
        dict(name="concat_nhwc", kind="concat_nhwc", dtype="fp16", batch=32, size=28, branches="64,96,128,32"),
        # Channels-last to channel-major with an odd image size: rows of 1225 elements, nothing aligned.
        dict(name="nchw_odd", kind="nchw", dtype="bf16", batch=64, channels=288, size=35),
        # A projection that reads the attention output [b, heads, seq, dim] as the matrix of its rows: full batch.
        dict(name="attn_out_large", kind="attn_out", batch=16, seq=512, heads=16, dim=64, n=4096, weight="kn"),
        # The output projection for one sequence (serving at batch 1), the weight kept [n, k] as linear layers keep it.
        dict(name="attn_out_one", kind="attn_out", batch=1, seq=512, heads=16, dim=64, n=1024, weight="nk"),
        # A QKV projection at a small batch whose product is stored split by heads.
        dict(name="qkv_proj", kind="qkv_proj", batch=4, seq=512, heads=12, dim=64),
        # A pointwise convolution that reads its channel-major activation directly and writes channels-last rows.
        dict(name="conv1x1", kind="conv1x1", batch=32, size=56, branches="256", n=512),
        # The same behind a channel concat: four branches gathered in the operand load.
        dict(name="conv1x1_concat", kind="conv1x1", batch=128, size=28, branches="64,96,128,32", n=256),
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(["tokens", "nhwc_pad", "qkv_split", "head_merge", "concat_nhwc", "nchw", "attn_out", "qkv_proj", "conv1x1"])
    while True:
        if kind == "tokens":
            c = dict(kind=kind, dtype=rng.choice(["fp32", "bf16"]), batch=_log(rng, 1, 64), channels=rng.choice([8, 12, 16, 24, 32]),
                     size=rng.choice([14, 16, 28, 32, 35]), pad=rng.choice([0, 1, 4, 8]))
        elif kind == "nhwc_pad":
            c = dict(kind=kind, dtype=rng.choice(["bf16", "fp32"]), batch=_log(rng, 1, 128), channels=rng.choice([48, 64, 75, 96, 256, 512, 1000, 2048]),
                     size=rng.choice([7, 14, 17, 28, 35, 56, 57, 112]), pad=rng.choice([0, 1, 1, 2]))
        elif kind == "nchw":
            c = dict(kind=kind, dtype=rng.choice(["bf16", "fp32"]), batch=_log(rng, 1, 128), channels=rng.choice([48, 64, 96, 100, 256, 288, 768, 2048]),
                     size=rng.choice([7, 14, 17, 28, 35, 55, 56]))
        elif kind in ("qkv_split", "head_merge"):
            c = dict(kind=kind, dtype=rng.choice(["bf16", "fp16", "fp32"]), batch=_log(rng, 1, 64), seq=_log(rng, 33, 2048),
                     heads=rng.choice([8, 12, 16, 20]), dim=rng.choice([32, 64, 80, 128]))
        elif kind == "concat_nhwc":
            c = dict(kind=kind, dtype=rng.choice(["fp16", "bf16", "fp32"]), batch=_log(rng, 1, 128), size=rng.choice([8, 14, 17, 28, 56]),
                     branches=",".join(str(rng.choice([24, 32, 64, 96, 128, 192])) for _ in range(rng.randint(2, 4))))
        elif kind == "attn_out":
            c = dict(kind=kind, batch=_log(rng, 1, 16), seq=_log(rng, 33, 2048), heads=rng.choice([8, 12, 16, 20]), dim=rng.choice([32, 64, 64, 80, 128]),
                     n=rng.choice([512, 768, 1000, 1024, 2048, 4096]), weight=rng.choice(["kn", "nk"]))
        elif kind == "qkv_proj":
            c = dict(kind=kind, batch=_log(rng, 1, 16), seq=_log(rng, 33, 1024), heads=rng.choice([8, 12, 16]), dim=rng.choice([32, 64, 64, 80]))
        else:
            c = dict(kind=kind, batch=_log(rng, 1, 128), size=rng.choice([8, 12, 28, 28, 56]),
                     branches=",".join(str(rng.choice([32, 64, 96, 128, 256])) for _ in range(rng.randint(1, 4))), n=rng.choice([64, 120, 128, 256, 512]))
        w = work(c)
        if 1e5 < w["bytes"] < 1.2e8 and w["flops"] < 4e10:
            return c


def _channels(case):
    return [int(c) for c in case["branches"].split(",")]


def _dims(case):
    """(source shapes, operator list, output shape) of a layout chain, or of the A operand of a product."""
    k, b = case["kind"], case["batch"]
    if k == "tokens":
        s, c = case["size"], case["channels"]
        lo, hi = s * s // 8, s * s - s * s // 8
        return [(b, c, s, s)], [("transpose", (0, 2, 3, 1)), ("reshape", (b, s * s, c)), ("slice", 1, lo, hi, 1),
                                ("pad", (0, 0, 0), (0, 0, case["pad"]), 0)], (b, hi - lo, c + case["pad"])
    if k == "nhwc_pad":
        s, c, p = case["size"], case["channels"], case["pad"]
        return [(b, c, s, s)], [("transpose", (0, 2, 3, 1)), ("pad", (0, p, p, 0), (0, p, p, 0), 0)], (b, s + 2 * p, s + 2 * p, c)
    if k == "nchw":
        s, c = case["size"], case["channels"]
        return [(b, s, s, c)], [("transpose", (0, 3, 1, 2))], (b, c, s, s)
    if k == "head_merge":
        n, h, d = case["seq"], case["heads"], case["dim"]
        return [(b, h, n, d)], [("transpose", (0, 2, 1, 3)), ("reshape", (b, n, h * d))], (b, n, h * d)
    if k == "concat_nhwc":
        s, cs = case["size"], _channels(case)
        return [(b, c, s, s) for c in cs], [("concat", 1), ("transpose", (0, 2, 3, 1))], (b, s, s, sum(cs))
    if k == "attn_out":
        n, h, d = case["seq"], case["heads"], case["dim"]
        return [(b, h, n, d)], [("transpose", (0, 2, 1, 3)), ("reshape", (b * n, h * d))], (b * n, h * d)
    if k == "qkv_proj":
        m, kk = b * case["seq"], case["heads"] * case["dim"]
        return [(m, kk)], [], (m, kk)
    s, cs = case["size"], _channels(case)   # conv1x1
    join = [("concat", 1)] if len(cs) > 1 else []
    return [(b, c, s, s) for c in cs], join + [("transpose", (0, 2, 3, 1)), ("reshape", (b * s * s, sum(cs)))], (b * s * s, sum(cs))


def _volume(shape):
    v = 1
    for e in shape:
        v *= e
    return v


def _columns(case):
    return 3 * case["heads"] * case["dim"] if case["kind"] == "qkv_proj" else case["n"]


def work(case):
    if case["kind"] in ("attn_out", "qkv_proj", "conv1x1"):
        m, k = _dims(case)[2]
        n = _columns(case)
        return {"bytes": 2 * (m * k + k * n + m * n), "flops": 2 * m * n * k}
    es = torch.empty(0, dtype=DTYPES[case["dtype"]]).element_size()
    if case["kind"] == "qkv_split":
        return {"bytes": 2 * es * case["batch"] * case["seq"] * 3 * case["heads"] * case["dim"], "flops": 0}
    srcs, _, out = _dims(case)
    read = sum(_volume(s) for s in srcs)
    if case["kind"] == "tokens":   # the cropped positions are not needed
        read = out[0] * out[1] * case["channels"]
    return {"bytes": es * (read + _volume(out)), "flops": 0}


def tolerance(case):
    # Copies are bit for bit.  A product of bf16 operands summed in fp32 and rounded once to bf16 lies 1.7e-3 from the
    # 64-bit one; about four times that.
    return {"rel": 7e-3} if case["kind"] in ("attn_out", "qkv_proj", "conv1x1") else "exact"


def _inputs(case, seed):
    """The input tensors of a case, from the seed alone: activations N(0, 1) or uniform, weights N(0, 0.02)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = DTYPES[case.get("dtype", "bf16")]

    def normal(shape, std=1.0):
        return torch.randn(shape, device="cuda", generator=g).mul_(std).to(dt)

    if case["kind"] == "qkv_split":
        return [normal((case["batch"], case["seq"], 3 * case["heads"] * case["dim"]))], None
    srcs, _, out = _dims(case)
    if case["kind"] == "concat_nhwc":
        return [torch.rand(s, device="cuda", generator=g).mul_(2).sub_(1).to(dt) for s in srcs], None
    x = [normal(s) for s in srcs]
    if case["kind"] not in ("attn_out", "qkv_proj", "conv1x1"):
        return x, None
    k, n = out[1], _columns(case)
    return x, normal((n, k) if case.get("weight") == "nk" else (k, n), 0.02)


def prepare(case, seed):
    x, w = _inputs(case, seed)
    kind, dt = case["kind"], x[0].dtype
    es = x[0].element_size()
    state = {"kind": kind, "x": x, "w": w}
    if kind == "qkv_split":
        b, s, h, d = case["batch"], case["seq"], case["heads"], case["dim"]
        chain = [("reshape", (b, s, 3, h, d)), ("transpose", (2, 0, 3, 1, 4))]
        state["maps"] = [B.amap_compose([tuple(x[0].shape)], es, chain + [("slice", 0, t, t + 1, 1), ("reshape", (b, h, s, d))])
                         for t in range(3)]
        state["out"] = [torch.empty((b, h, s, d), dtype=dt, device="cuda") for _ in range(3)]
        return state
    srcs, ops, out = _dims(case)
    state["map"] = B.amap_compose(srcs, es, ops)
    if w is None:
        state["out"] = torch.empty(out, dtype=dt, device="cuda")
        return state
    m, n = out[0], _columns(case)
    if case.get("weight") == "nk":
        state["w_map"] = B.amap_compose([tuple(w.shape)], 2, [("transpose", (1, 0))])
    if kind == "qkv_proj":
        b, s, h, d = case["batch"], case["seq"], case["heads"], case["dim"]
        state["out_map"] = B.amap_compose([(m, n)], 2, [("reshape", (b, s, 3, h, d)), ("transpose", (2, 0, 3, 1, 4))])
        state["out"] = torch.empty((3, b, h, s, d), dtype=dt, device="cuda")
    else:
        state["out"] = torch.empty((m, n), dtype=dt, device="cuda")
    return state


def run(state):
    kind, x, out = state["kind"], state["x"], state["out"]
    if kind == "qkv_split":
        return device.execute_multi(state["maps"], x, out)
    if state["w"] is None:
        return device.execute(state["map"], x, out)
    w = state["w"]
    if len(x) > 1:
        B.amap_gemm_gather([t.data_ptr() for t in x], state["map"], w.data_ptr(), None, w.shape[1], None, out.data_ptr(), device.current_stream())
        return out
    if "w_map" in state:
        B.amap_gemm_mapped(x[0].data_ptr(), state["map"], w.data_ptr(), state["w_map"], None, out.data_ptr(), device.current_stream())
        return out
    return device.gemm_fused(x[0], state["map"], w, out, out_map=state.get("out_map"))


def exact(case, seed):
    if case["kind"] not in ("attn_out", "qkv_proj", "conv1x1"):
        return None   # copies: nothing is computed
    x, w = _inputs(case, seed)
    w = w.double()
    if case.get("weight") == "nk":
        w = w.t().contiguous()
    if case["kind"] == "attn_out":
        a = x[0].permute(0, 2, 1, 3)
    elif case["kind"] == "conv1x1":
        a = torch.cat(x, 1).permute(0, 2, 3, 1)
    else:
        a = x[0]
    y = a.reshape(-1, w.shape[0]).double() @ w
    if case["kind"] == "qkv_proj":
        b, s, h, d = case["batch"], case["seq"], case["heads"], case["dim"]
        y = y.reshape(b, s, 3, h, d).permute(2, 0, 3, 1, 4).contiguous()
    return y
