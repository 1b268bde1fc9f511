"""The work that a program has this library do, as timed cases: one GPU's share of a fully-connected
layer under 3D tensor parallelism, called through the public entry points on buffers that the program
owns.

A case gives the problem statement (grid, global token count T, in-features K, out-features N; this GPU
sits at the grid's origin) and how it is called:

  how = "forward"    axo_fc_fwd alone: evaluation, or the forward half of a step whose backward comes later
  how = "calls"      the products of a layer one call at a time, as a training loop makes them that puts a
                     collective behind every product: forward, data gradient, weight gradient, and the
                     bias gradient where db is set
  how = "step"       the chain entry point axo_layer_step over `layers` (a single layer, or a transformer
                     block's four: qkv, attention output, MLP up with bias + GELU, MLP down), K the hidden size
  how = "step_ext"   axo_layer_step_ext, one layer with the backward-side extras that are switched on
  how = "bias_grad"  axo_bias_grad_ws alone

  epi   forward epilogue (0 none, 1 bias, 2 bias + tanh GELU, 3 bias + erf GELU)
  act   data gradient through the GELU of the layer below (0 plain, 2 tanh form, 3 erf form)
  acc   weight gradient accumulated into an fp32 master gradient
  db    bias gradient wanted (accumulated where acc is)
  gap   elements between the end of a matrix row (rounded up to 8) and the next row: shards addressed in
        place inside wider matrices

Inputs: activations and output gradients N(0, 1), weights and biases N(0, 0.02), as at initialisation of
the networks the library is for; bf16, accumulators fp32.
"""
import math

import torch

import paper_2305_13525_amd as axo

DEV = "cuda:0"
SIGMA_W = 0.02


def _case(name, how, T, K, N, grid=(1, 1, 1), epi=0, act=0, acc=False, db=False, gap=0, layers="one"):
    return {"name": name, "how": how, "T": T, "K": K, "N": N, "gx": grid[0], "gy": grid[1], "gz": grid[2],
            "epi": epi, "act": act, "acc": acc, "db": db, "gap": gap, "layers": layers}


def listed():
    return [
        # the smallest call: a 256 x 256 x 256 shard of a 512 x 512 x 512 layer on 8 GPUs; nothing but latency
        _case("forward_smallest", "forward", 512, 512, 512, (2, 2, 2)),
        # a small layer, one call per product (the repository's smallest configuration)
        _case("calls_small", "calls", 512, 1024, 1024),
        # a short batch on a mid-size layer: fewer tokens than a tile has rows, the weights are what is read
        _case("calls_few_tokens", "calls", 96, 2048, 6144, epi=2, act=2),
        # nothing is a multiple of anything; rows padded to the 16 bytes that the interface asks for
        _case("calls_odd", "calls", 1001, 1027, 515, epi=1, act=3, gap=8),
        # a ragged mid-size shard: multiples of 8 and no more
        _case("calls_ragged", "calls", 4000, 2000, 6000, epi=3),
        # attention output projection of a 12288-wide model on 64 x 4 GPUs, fp32 master gradient and bias
        # gradient, product by product
        _case("calls_attn_out_master", "calls", 16384, 12288, 12288, (8, 8, 4), epi=1, acc=True, db=True),
        # qkv projection of a 4096-wide model on 16 GPUs, the chain entry point
        _case("step_qkv", "step", 16384, 4096, 12288, (2, 2, 4)),
        # the same layer's whole local step with every backward-side extra
        _case("step_ext_qkv", "step_ext", 16384, 4096, 12288, (2, 2, 4), epi=1, act=2, acc=True, db=True),
        # MLP up projection of an 8192-wide model on 64 GPUs with bias + GELU, product by product: large GEMMs
        _case("calls_mlp_up", "calls", 32768, 8192, 32768, (4, 2, 8), epi=2),
        # one block of a 12288-wide model on 256 GPUs: twelve small products in one call
        _case("block_12288", "step", 16384, 12288, 0, (8, 8, 4), layers="block"),
        # one block of a 7168-wide (20B) model on 16 GPUs: the largest
        _case("block_7168", "step", 32768, 7168, 0, (2, 2, 4), layers="block"),
        # the bias gradient on its own: column sums, memory bound
        _case("bias_grad_qkv", "bias_grad", 16384, 4096, 12288, (2, 2, 4)),
    ]


def _log_size(rng, lo, hi):
    """A size spread over the logarithm of [lo, hi]: a third of them any number, a third multiples of 8, the
    rest multiples of 128."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    unit = rng.choice((1, 8, 128))
    return max(1, lo if v < lo else int(v / unit + 0.5) * unit or unit)


def draw(rng):
    how = rng.choice(("forward", "calls", "calls", "calls", "step", "step_ext", "bias_grad"))
    gap = rng.choice((0, 0, 0, 8, 64, 4096))
    if how == "step" and rng.random() < 0.5:  # a block of four layers
        gx, gy, gz = rng.choice(((1, 1, 1), (2, 2, 4), (2, 4, 2), (4, 4, 4), (8, 8, 4)))
        hidden = 64 * rng.randint(4, 28) * max(gx, gy)
        tokens = rng.randint(64, 8192) * gz
        return {k: v for k, v in _case("", "step", tokens, hidden, 0, (gx, gy, gz), gap=gap, layers="block").items()
                if k != "name"}
    while True:
        m, k, n = _log_size(rng, 1, 16384), _log_size(rng, 32, 16384), _log_size(rng, 32, 16384)
        if 2.0 * m * k * n <= 4e11:  # a layer's three products stay well below the largest listed case
            break
    gx, gy, gz = (1, 1, 1) if how == "bias_grad" else rng.choice(((1, 1, 1), (2, 2, 2), (4, 2, 8)))
    c = _case("", how, m * gz, k * gx, n * gy, (gx, gy, gz), gap=gap)
    if how in ("forward", "calls", "step", "step_ext"):
        c["epi"] = rng.randint(0, 3)
    if how in ("calls", "step_ext"):
        c["act"], c["acc"], c["db"] = rng.choice((0, 2, 3)), rng.random() < 0.4, rng.random() < 0.4
    del c["name"]
    return c


def _problems(case):
    """(problem, forward epilogue) of each layer."""
    grid = (case["gx"], case["gy"], case["gz"])
    mk = lambda k, n: axo.Problem.make(grid, (0, 0, 0), case["T"], k, n)  # noqa: E731
    if case["layers"] == "block":
        h = case["K"]
        return [(mk(h, 3 * h), 0), (mk(h, h), 0), (mk(h, 4 * h), 2), (mk(4 * h, h), 0)]
    return [(mk(case["K"], case["N"]), case["epi"])]


def _shards(case):
    """(M, Kl, Nl, epilogue) of each layer."""
    gx, gy, gz = case["gx"], case["gy"], case["gz"]
    return [(p.T // gz, p.K // gx, p.N // gy, e) for p, e in _problems(case)]


def _inputs(case, seed):
    """The bf16 inputs of each layer (and the fp32 gradients so far), made on the GPU from the seed alone."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)

    def normal(rows, cols, sigma=1.0, dtype=torch.bfloat16):
        pitch = (cols + 7) // 8 * 8 + case["gap"]
        a = torch.empty((rows, pitch), dtype=dtype, device=DEV)
        a.normal_(0.0, sigma, generator=gen)
        return a[:, :cols]

    layers = []
    for m, k, n, epi in _shards(case):
        t = {}
        if case["how"] != "bias_grad":
            t["X"], t["W"] = normal(m, k), normal(k, n, SIGMA_W)
        if epi:
            t["bias"] = normal(1, n, SIGMA_W)[0]
        if case["how"] != "forward":
            t["dY"] = normal(m, n)
        if case["act"]:
            t["pre"] = normal(m, k)
        if case["acc"]:
            t["dW32"] = normal(k, n, 10.0, torch.float32)  # what earlier micro-batches left
        if case["db"] or case["how"] == "bias_grad":
            t["db"] = normal(1, n, 10.0, torch.float32)[0]
        layers.append(t)
    return layers


def _pitched(rows, cols, gap):
    return torch.zeros((rows, (cols + 7) // 8 * 8 + gap), dtype=torch.bfloat16, device=DEV)[:, :cols]


def _ptr(t):
    return None if t is None else t.data_ptr()


def prepare(case, seed):
    how, layers = case["how"], _inputs(case, seed)
    for t, (m, k, n, epi), (p, _) in zip(layers, _shards(case), _problems(case)):
        t["p"], t["epi"] = p, epi
        if how != "bias_grad":
            t["Y"] = _pitched(m, n, case["gap"])
        if how in ("calls", "step", "step_ext"):
            t["dX"] = _pitched(m, k, case["gap"])
            if not case["acc"]:
                t["dW"] = _pitched(k, n, case["gap"])
        if (case["db"] and how == "calls") or how == "bias_grad":
            t["db_ws_bytes"] = axo.axo_bias_grad_workspace_bytes(p)
            t["db_ws"] = torch.zeros(max(16, t["db_ws_bytes"]), dtype=torch.uint8, device=DEV)
    state = {"case": case, "layers": layers, "stream": torch.cuda.current_stream().cuda_stream}
    ops = {"forward": (axo.AXO_OP_FWD,), "bias_grad": ()}.get(how, (axo.AXO_OP_FWD, axo.AXO_OP_DGRAD, axo.AXO_OP_WGRAD))
    need = max([axo.axo_workspace_bytes(t["p"], op) for t in layers for op in ops] + [0])
    state["ws_bytes"] = need
    state["ws"] = torch.zeros(need, dtype=torch.uint8, device=DEV) if need else None
    if how in ("step", "step_ext"):
        ld = lambda t: 0 if t is None else t.stride(0)  # noqa: E731
        state["structs"] = [axo.Layer(t["p"], t["epi"], 0, _ptr(t["X"]), ld(t["X"]), _ptr(t["W"]), ld(t["W"]), _ptr(t.get("bias")),
                                      _ptr(t["Y"]), ld(t["Y"]), _ptr(t["dY"]), ld(t["dY"]), _ptr(t["dX"]), ld(t["dX"]),
                                      _ptr(t.get("dW")), ld(t.get("dW"))) for t in layers]
        if how == "step_ext":
            state["structs"] = [axo.LayerExt.make(s, _ptr(t.get("pre")), ld(t.get("pre")), case["act"], _ptr(t.get("dW32")),
                                                  ld(t.get("dW32")), _ptr(t.get("db")), int(case["db"] and case["acc"]))
                                for s, t in zip(state["structs"], layers)]
    return state


def run(state):
    case, how, stream = state["case"], state["case"]["how"], state["stream"]
    ws, ws_bytes = _ptr(state["ws"]), state["ws_bytes"]
    if how == "step":
        axo.axo_layer_step(state["structs"], ws, ws_bytes, stream)
    elif how == "step_ext":
        axo.axo_layer_step_ext(state["structs"], ws, ws_bytes, stream)
    elif how == "bias_grad":
        t = state["layers"][0]
        axo.axo_bias_grad_ws(t["p"], t["dY"].data_ptr(), t["dY"].stride(0), t["db"].data_ptr(), 0, t["db_ws"].data_ptr(),
                             t["db_ws_bytes"], stream)
        return [t["db"]]
    else:
        t = state["layers"][0]
        p, X, W, Y = t["p"], t["X"], t["W"], t["Y"]
        axo.axo_fc_fwd(p, X.data_ptr(), X.stride(0), W.data_ptr(), W.stride(0), _ptr(t.get("bias")), t["epi"],
                       Y.data_ptr(), Y.stride(0), ws, ws_bytes, stream)
        if how == "calls":
            dY, dX = t["dY"], t["dX"]
            if case["act"]:
                axo.axo_fc_dgrad_act(p, dY.data_ptr(), dY.stride(0), W.data_ptr(), W.stride(0), t["pre"].data_ptr(),
                                     t["pre"].stride(0), case["act"], dX.data_ptr(), dX.stride(0), ws, ws_bytes, stream)
            else:
                axo.axo_fc_dgrad(p, dY.data_ptr(), dY.stride(0), W.data_ptr(), W.stride(0), dX.data_ptr(), dX.stride(0),
                                 ws, ws_bytes, stream)
            if case["acc"]:
                axo.axo_fc_wgrad_acc(p, X.data_ptr(), X.stride(0), dY.data_ptr(), dY.stride(0), t["dW32"].data_ptr(),
                                     t["dW32"].stride(0), ws, ws_bytes, stream)
            else:
                axo.axo_fc_wgrad(p, X.data_ptr(), X.stride(0), dY.data_ptr(), dY.stride(0), t["dW"].data_ptr(),
                                 t["dW"].stride(0), ws, ws_bytes, stream)
            if case["db"]:
                axo.axo_bias_grad_ws(p, dY.data_ptr(), dY.stride(0), t["db"].data_ptr(), int(case["acc"]),
                                     t["db_ws"].data_ptr(), t["db_ws_bytes"], stream)
    return [[t[k] for k in ("Y", "dX", "dW", "dW32", "db") if k in t] for t in state["layers"]]


def work(case):
    """Each input read once, each output written once (an accumulated gradient read and written)."""
    how, flops, elems2, elems4 = case["how"], 0.0, 0.0, 0.0
    for m, k, n, epi in _shards(case):
        if how == "bias_grad":
            flops, elems2, elems4 = flops + m * n, elems2 + m * n, elems4 + n
            continue
        products = 1 if how == "forward" else 3
        flops += products * 2.0 * m * k * n
        elems2 += m * k + k * n + m * n + (n if epi else 0)  # X, W, Y
        if products == 3:
            elems2 += m * n + m * k + (m * k if case["act"] else 0)  # dY, dX, pre
            if case["acc"]:
                elems4 += 2 * k * n
            else:
                elems2 += k * n
            if case["db"]:
                elems4 += n * (2 if case["acc"] else 1)
                flops += m * n
    return {"bytes": 2.0 * elems2 + 4.0 * elems4, "flops": flops}


def tolerance(case):
    if case["how"] == "bias_grad":  # fp32 sums of bf16 values: 4e-8 measured against 64 bits, and sums in another order differ
        # from these by about twice that; up to four times as many rows are drawn
        return {"rel": 3e-7, "max": 3e-6}
    # One rounding of an fp32 sum to bf16: 1.66e-3 from the 64-bit value in the 2-norm, at most half a step
    # (2^-8 of the value) in one element, one step where the sum lies next to a rounding boundary.
    return {"rel": 6e-3, "max": 2e-2}


def _gelu(v, form):
    return torch.nn.functional.gelu(v, approximate="tanh" if form == 2 else "none")


def _dgelu(v, form):
    if form == 3:
        return 0.5 * (1.0 + torch.erf(v / math.sqrt(2.0))) + v * torch.exp(-0.5 * v * v) / math.sqrt(2.0 * math.pi)
    c = math.sqrt(2.0 / math.pi)
    th = torch.tanh(c * (v + 0.044715 * v ** 3))
    return 0.5 * (1.0 + th) + 0.5 * v * (1.0 - th * th) * c * (1.0 + 3.0 * 0.044715 * v * v)


def exact(case, seed):
    out = []
    for t, (m, k, n, epi) in zip(_inputs(case, seed), _shards(case)):
        d = {key: v.double() for key, v in t.items()}
        if case["how"] == "bias_grad":
            return [d["dY"].sum(0)]
        y = d["X"] @ d["W"]
        if epi:
            y += d["bias"]
        got = [_gelu(y, epi) if epi >= 2 else y]
        if case["how"] != "forward":
            dx = d["dY"] @ d["W"].t()
            got.append(dx * _dgelu(d["pre"], case["act"]) if case["act"] else dx)
            dw = d["X"].t() @ d["dY"]
            got.append(dw + d["dW32"] if case["acc"] else dw)
            if case["db"]:
                db = d["dY"].sum(0)
                got.append(db + d["db"] if case["acc"] else db)
        out.append(got)
    return out
