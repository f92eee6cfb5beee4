"""The work that a program using this library has it do: products, convolutions and recurrent layers of BCR-pruned
weights, through the package's public entry points.

A case names its kind ("spmv", "group", "rnn_step", "rnn_seq", "spmm", "conv"), the element type, the block size
(br x bc), what every block keeps (kr rows and kc columns, or "mixed": the fractions 1/8, 1/4 and 1/2 drawn per block
and direction) and the sizes of its kind.  Weights, masks, plans and state buffers are made in prepare(), as an inference
program makes them once; run() is one pass: a call (or the few calls of a small stack of layers) on inputs that are
already on the GPU.
"""
import math

import numpy as np
import torch

import paper_2108_11033_amd as g
from paper_2108_11033_amd import binding

TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZE = {"f32": 4, "f16": 2, "bf16": 2}


def listed():
    return [
        # One gate product of an LSTM layer with 1024 units and inputs, one vector: the smallest call, where launch and
        # latency count (a server answering one request at a time).
        dict(name="spmv_gates_b1", kind="spmv", dtype="f16", M=4096, K=2048, br=32, bc=32, kr=8, kc=12, mixed=False, batch=1),
        # A fully connected layer whose blocks were pruned at different rates, five vectors at once.
        dict(name="spmv_fc_mixed_b5", kind="spmv", dtype="bf16", M=4096, K=4096, br=32, bc=32, kr=0, kc=0, mixed=True, batch=5),
        # 64 gate matrices of that size, each with a vector of its own, in one launch: models served side by side.
        dict(name="spmv_group_64", kind="group", dtype="f16", M=4096, K=2048, br=32, bc=32, kr=8, kc=12, mixed=False, batch=1, count=64),
        # One time step of a two-layer GRU of 1024 units at batch 32, 160 input features: streaming speech recognition.
        dict(name="gru_step_b32", kind="rnn_step", cell="gru", dtype="f16", H=1024, I=160, layers=2, br=32, bc=32, kr=8, kc=12,
             mixed=False, batch=32),
        # A whole utterance of 64 frames for eight callers at once through an LSTM layer.
        dict(name="lstm_sequence_b8", kind="rnn_seq", cell="lstm", dtype="f16", H=1024, I=1024, br=32, bc=32, kr=8, kc=12, T=64, batch=8),
        # A 3x3 layer of 128 -> 256 channels on a 56x56 map as a product with the im2col matrix, in fp32.
        dict(name="spmm_f32_layer", kind="spmm", dtype="f32", M=256, K=1152, N=3136, br=16, bc=32, kr=8, kc=8, mixed=False),
        # The ordinary half-precision layer: 256 -> 256 channels, 3x3, 56x56.
        dict(name="spmm_f16_layer", kind="spmm", dtype="f16", M=256, K=2304, N=3136, br=16, bc=32, kr=8, kc=8, mixed=False),
        # The last stage of an image network, 512 channels on three 7x7 maps: 147 columns, rows that are not aligned.
        dict(name="spmm_f16_ragged", kind="spmm", dtype="f16", M=512, K=4608, N=147, br=16, bc=32, kr=8, kc=8, mixed=False),
        # The largest product: 512 channels, 3x3, a batch of eight 56x56 maps, blocks pruned at different rates.
        dict(name="spmm_bf16_large", kind="spmm", dtype="bf16", M=512, K=4608, N=25088, br=32, bc=32, kr=0, kc=0, mixed=True),
        # Three chained 3x3 layers of 512 channels on one 14x14 map with bias and rectifier: the deep stage of a
        # classifier answering one image.
        dict(name="conv_chain_14", kind="conv", form="chain", depth=3, dtype="f16", out="f16", cin=512, cout=512, h=14, w=14, k=3,
             stride=1, batch=1, br=16, bc=32, kr=8, kc=8, mixed=False),
        # The entry of a residual stage on four 56x56 maps (3x3 at stride 2, 3x3, and the 1x1 shortcut at stride 2),
        # pruned in 4x16 blocks.
        dict(name="conv_residual_4x16", kind="conv", form="residual", depth=3, dtype="f16", out="f16", cin=128, cout=256, h=56, w=56,
             k=3, stride=2, batch=4, br=4, bc=16, kr=2, kc=4, mixed=False),
        # 512 channels, 3x3, on a batch of eight 56x56 maps, straight from the feature maps.
        dict(name="conv_large", kind="conv", form="chain", depth=1, dtype="bf16", out="bf16", cin=512, cout=512, h=56, w=56, k=3,
             stride=1, batch=8, br=32, bc=32, kr=0, kc=0, mixed=True),
    ]


# ---------------------------------------------------------------------------------------------------- drawn cases
def _log(rng, lo, hi):
    """An integer of [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _fc_blocks(rng):
    """Block size and kept counts of fully connected and recurrent layers."""
    br, bc, kr, kc = rng.choice([(32, 32, 8, 12), (32, 32, 8, 12), (32, 32, 8, 8), (32, 32, 16, 8), (16, 32, 4, 12), (8, 32, 4, 8),
                                 (32, 32, 10, 10)])
    mixed = rng.random() < 0.3
    return dict(br=br, bc=bc, kr=0 if mixed else kr, kc=0 if mixed else kc, mixed=mixed)


def _layer_blocks(rng):
    """The same for convolutional layers."""
    br, bc, kr, kc = rng.choice([(16, 32, 8, 8), (16, 32, 8, 8), (32, 32, 8, 16), (4, 16, 2, 4), (16, 16, 4, 8), (8, 16, 4, 4)])
    mixed = br >= 8 and rng.random() < 0.3
    return dict(br=br, bc=bc, kr=0 if mixed else kr, kc=0 if mixed else kc, mixed=mixed)


def draw(rng):
    most = max(_weight(c) for c in listed())
    while True:
        c = _draw(rng)
        if _weight(c) <= most:
            return c


def _weight(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 50)


def _draw(rng):
    kind = rng.choice(["spmv", "group", "rnn_step", "rnn_seq", "spmm", "spmm", "spmm", "conv", "conv", "conv"])
    half = rng.choice(["f16", "bf16"])
    if kind == "spmv":
        return dict(kind=kind, dtype=rng.choice(["f16", "bf16", "f32"]), M=32 * _log(rng, 8, 160), K=32 * _log(rng, 8, 128),
                    batch=rng.randint(1, 8), **_fc_blocks(rng))
    if kind == "group":
        c = dict(kind=kind, dtype=half, M=32 * _log(rng, 16, 128), K=32 * _log(rng, 16, 64), batch=rng.choice([1, 1, 2, 3, 4, 8]),
                 count=_log(rng, 4, 64), **_fc_blocks(rng))
        return c
    if kind == "rnn_step":
        H = 32 * _log(rng, 8, 64)
        return dict(kind=kind, cell=rng.choice(["lstm", "gru"]), dtype=half, H=H, I=32 * _log(rng, 2, H // 32), layers=rng.choice([1, 2]),
                    batch=_log(rng, 1, 64), **_fc_blocks(rng))
    if kind == "rnn_seq":
        # (the whole-sequence call takes uniformly pruned layers of at most 64 column blocks)
        H = 32 * _log(rng, 8, 32)
        kr, kc = rng.choice([(8, 12), (8, 8), (4, 16), (16, 8)])
        return dict(kind=kind, cell=rng.choice(["lstm", "gru"]), dtype=half, H=H, I=H if rng.random() < 0.5 else 32 * _log(rng, 2, 32),
                    T=_log(rng, 8, 128), batch=_log(rng, 1, 32), br=32, bc=32, kr=kr, kc=kc)
    if kind == "spmm":
        b = _layer_blocks(rng)
        N = _log(rng, 16, 25088)
        if rng.random() < 0.6:
            N = (N + 7) // 8 * 8
        return dict(kind=kind, dtype=rng.choice(["f16", "f16", "bf16", "bf16", "f32"]), M=32 * _log(rng, 2, 16), K=96 * _log(rng, 3, 48),
                    N=N, **b)
    b = _layer_blocks(rng)
    form = rng.choice(["chain", "chain", "residual"])
    side = _log(rng, 7, 112)
    k = 3 if form == "residual" else rng.choice([1, 3, 3, 3, 5])
    cin = 32 * _log(rng, 2, 16)
    depth = 3 if form == "residual" else rng.choice([1, 1, 2, 3])
    return dict(kind="conv", form=form, depth=depth, dtype=half, out=half if depth > 1 else rng.choice([half, "f32"]), cin=cin,
                cout=cin if rng.random() < 0.5 else 32 * _log(rng, 2, 16), h=side, w=side if rng.random() < 0.7 else _log(rng, 7, 112),
                k=k, stride=2 if form == "residual" else rng.choice([1, 1, 1, 2]), batch=_log(rng, 1, 8), **b)


# ---------------------------------------------------------------------------------------------------- inputs
FRACTIONS = (0.125, 0.25, 0.5)


def _mixed_counts(size):
    return [max(1, int(round(size * f))) for f in FRACTIONS]


def _keep(rng, nb, size, count, mixed):
    """Per block `count` (or a mixed count) of `size` indices, uniform without replacement: (ptr, ascending idx)."""
    counts = np.asarray(_mixed_counts(size))[rng.integers(0, 3, nb)] if mixed else np.full(nb, count)
    keys = rng.integers(0, 1 << 24, size=(nb, size), dtype=np.int32) * 64 + np.arange(size, dtype=np.int32)
    order = np.sort(keys, axis=1) % 64                       # a random permutation per block (block sides are at most 32)
    chosen = np.arange(size)[None, :] < counts[:, None]
    flags = np.zeros((nb, size), dtype=bool)
    np.put_along_axis(flags, order.astype(np.int64), chosen, axis=1)
    ptr = np.zeros(nb + 1, dtype=np.int32)
    np.cumsum(counts, out=ptr[1:])
    return ptr, np.nonzero(flags)[1].astype(np.uint16)


def _storage(values, dtype):
    """fp32 values in the storage type as the packer takes it (bf16: bit patterns)."""
    if dtype == "f32":
        return values
    if dtype == "f16":
        return values.astype(np.float16)
    return torch.from_numpy(values).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)


def _pack(rng, case, M, K, sigma, pool=None):
    """A packed M x K matrix; `pool`: normal values in storage type to cut the weights from."""
    br, bc = case["br"], case["bc"]
    nb = (M // br) * (K // bc)
    rows = _keep(rng, nb, br, case["kr"], case.get("mixed", False))
    cols = _keep(rng, nb, bc, case["kc"], case.get("mixed", False))
    if pool is None:
        W = _storage(rng.standard_normal((M, K), dtype=np.float32) * np.float32(sigma), case["dtype"])
    else:
        at = int(rng.integers(0, pool.size - M * K + 1))
        W = pool[at:at + M * K].reshape(M, K)
    return g.pack(W, case["dtype"], br, bc, rows[0], rows[1], cols[0], cols[1])


def _kept_share(case):
    if case.get("mixed"):
        return (sum(_mixed_counts(case["br"])) / 3 / case["br"]) * (sum(_mixed_counts(case["bc"])) / 3 / case["bc"])
    return case["kr"] * case["kc"] / (case["br"] * case["bc"])


def _normal(gen, shape, dtype, relu=False):
    x = torch.randn(shape, dtype=torch.float32, device="cuda", generator=gen)
    return (x.clamp_(min=0) if relu else x).to(TORCH[dtype])


def _conv_layers(case):
    """(cin, cout, h, w, kernel, stride, input: index of an earlier layer or -1) of the case's layers."""
    half = lambda n: (n + 1) // 2
    k, s, cin, cout, h, w = case["k"], case["stride"], case["cin"], case["cout"], case["h"], case["w"]
    if case["form"] == "residual":
        return [(cin, cout, h, w, k, s, -1), (cout, cout, half(h), half(w), k, 1, 0), (cin, cout, h, w, 1, s, -1)]
    layers = [(cin, cout, h, w, k, s, -1)]
    for i in range(1, case["depth"]):
        h, w = (half(h), half(w)) if layers[-1][5] == 2 else (h, w)
        layers.append((cout, cout, h, w, k, 1, i - 1))
    return layers


def prepare(case, seed):
    rng = np.random.default_rng([20210811, int(seed)])
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    kind, dt = case["kind"], case["dtype"]
    s = {"case": case, "stream": torch.cuda.current_stream()}
    empty = lambda *shape: torch.empty(shape, dtype=torch.float32, device="cuda")
    zeros = lambda shape, d: torch.zeros(shape, dtype=d, device="cuda")
    if kind in ("spmv", "spmm"):
        n = case["batch"] if kind == "spmv" else case["N"]
        s["A"] = _pack(rng, case, case["M"], case["K"], 0.02)
        s["x"] = _normal(gen, (case["K"], n), dt, relu=kind == "spmm")
        s["y"] = empty(case["M"], n)
    elif kind == "group":
        M, K, n = case["M"], case["K"], case["count"]
        pool = _storage(rng.standard_normal(M * K + 65536, dtype=np.float32) * np.float32(0.02), dt)
        s["G"] = binding.group([_pack(rng, case, M, K, 0.02, pool) for _ in range(n)])
        s["x"] = _normal(gen, (n, K, case["batch"]), dt)
        s["y"] = empty(n, M, case["batch"])
    elif kind == "rnn_step":
        H, b = case["H"], case["batch"]
        s["turn"], s["layers"] = 0, []
        for layer in range(case["layers"]):
            I = case["I"] if layer == 0 else H
            if case["cell"] == "lstm":
                # [x; h] of this step and of the next; the layer above reads h where the layer below writes a copy of it
                p = {"A": _pack(rng, case, 4 * H, I + H, 0.07), "xh": [_normal(gen, (I + H, b), dt) for _ in range(2)],
                     "gates": empty(4 * H, b), "bias": torch.randn(4 * H, device="cuda", generator=gen) * 0.1,
                     "c": zeros((H, b), torch.float32), "h32": empty(H, b)}
            else:
                p = {"Ai": _pack(rng, case, 3 * H, I, 0.07), "Ah": _pack(rng, case, 3 * H, H, 0.07), "gi": empty(3 * H, b),
                     "gh": empty(3 * H, b), "bi": torch.randn(3 * H, device="cuda", generator=gen) * 0.1,
                     "bh": torch.randn(3 * H, device="cuda", generator=gen) * 0.1, "h32": zeros((H, b), torch.float32),
                     "h": [zeros((H, b), TORCH[dt]) for _ in range(2)]}
            p["I"] = I
            s["layers"].append(p)
        if case["cell"] == "gru":
            s["x"] = _normal(gen, (case["I"], b), dt)
    elif kind == "rnn_seq":
        H, I, b, T = case["H"], case["I"], case["batch"], case["T"]
        if case["cell"] == "lstm":
            s["A"] = _pack(rng, case, 4 * H, I + H, 0.07)
            s["bias"] = torch.randn(4 * H, device="cuda", generator=gen) * 0.1
        else:
            s["A"], s["Ah"] = _pack(rng, case, 3 * H, I, 0.07), _pack(rng, case, 3 * H, H, 0.07)
            s["bias"], s["bias_h"] = (torch.randn(3 * H, device="cuda", generator=gen) * 0.1 for _ in range(2))
        s["xs"] = _normal(gen, (T * b, I), dt)
        s["h0"] = zeros((b, H), TORCH[dt])
        s["state"] = zeros((b, H), torch.float32)
        s["hs"] = torch.empty((T * b, H), dtype=TORCH[dt], device="cuda")
        s["status"] = zeros((1,), torch.int32)
    else:
        b = case["batch"]
        s["x"] = _normal(gen, (b, case["cin"], case["h"], case["w"]), dt, relu=True)
        s["layers"] = []
        for (ci, co, h, w, k, st, src) in _conv_layers(case):
            K = ci * k * k
            A = _pack(rng, case, co, K, math.sqrt(2.0 / (K * _kept_share(case))))
            plan = g.ConvPlan(A, ci, h, w, k, k, st)
            out = torch.empty((b, co) + plan.out_hw, dtype=TORCH[case["out"]], device="cuda")
            s["layers"].append({"plan": plan, "src": src, "out": out, "bias": torch.randn(co, device="cuda", generator=gen) * 0.1,
                                "in_stride": ci * h * w, "hw": plan.out_hw[0] * plan.out_hw[1], "co": co})
    return s


# ---------------------------------------------------------------------------------------------------- one pass
def run(s):
    case, stream = s["case"], s["stream"]
    kind = case["kind"]
    if kind == "spmv":
        b = case["batch"]
        g.spmv(s["A"], s["x"], b, b, s["y"], b, stream)
        return s["y"]
    if kind == "spmm":
        n = case["N"]
        g.spmm(s["A"], s["x"], n, n, s["y"], n, stream)
        return s["y"]
    if kind == "group":
        b = case["batch"]
        g.spmv_batched(s["G"], s["x"], case["K"] * b, b, b, s["y"], case["M"] * b, b, stream)
        return s["y"]
    if kind == "rnn_step":
        b, H, now = case["batch"], case["H"], s["turn"]
        s["turn"] = 1 - now
        if case["cell"] == "lstm":
            for i, p in enumerate(s["layers"]):
                if i:
                    p["xh"][now][:H].copy_(s["layers"][i - 1]["h32"])
                g.lstm_step(p["A"], p["xh"][now], b, b, p["gates"], b, p["bias"], p["c"], b, p["xh"][1 - now][p["I"]:], b, p["h32"], b,
                            stream)
            return [[p["h32"], p["c"]] for p in s["layers"]]
        x, ldx = s["x"], b
        for p in s["layers"]:
            g.gru_step(p["Ai"], p["Ah"], x, ldx, p["h"][now], b, b, p["gi"], b, p["gh"], b, p["bi"], p["bh"], p["h32"], b,
                       p["h"][1 - now], b, stream)
            x = p["h"][1 - now]
        return [p["h32"] for p in s["layers"]]
    if kind == "rnn_seq":
        H, I, b, T = case["H"], case["I"], case["batch"], case["T"]
        if case["cell"] == "lstm":
            g.lstm_sequence_batch(s["A"], s["xs"], I, T, b, s["bias"], s["h0"], s["state"], s["hs"], H, None, 0, s["status"], 0, stream)
        else:
            g.gru_sequence_batch(s["A"], s["Ah"], s["xs"], I, T, b, s["bias"], s["bias_h"], s["h0"], s["state"], s["hs"], H, None, 0,
                                 s["status"], 0, stream)
        return [s["hs"], s["state"], s["status"]]
    b = case["batch"]
    for p in s["layers"]:
        x = s["x"] if p["src"] < 0 else s["layers"][p["src"]]["out"]
        g.conv2d_plan(p["plan"], x, b, p["in_stride"], p["bias"], True, p["out"], case["out"], p["hw"], p["co"] * p["hw"], stream)
    return [p["out"] for p in s["layers"][1:]] if case["form"] == "residual" else s["layers"][-1]["out"]


# ---------------------------------------------------------------------------------------------------- what a pass needs
def _matrix(case, M, K):
    """(bytes, kept weights) of a packed matrix: the kept values and, per block, its kept-row and kept-column sets as bits."""
    nnz = M * K * _kept_share(case)
    blocks = (M // case["br"]) * (K // case["bc"])
    return nnz * SIZE[case["dtype"]] + blocks * (case["br"] + case["bc"]) / 8, nnz


def work(case):
    kind, esz = case["kind"], SIZE[case["dtype"]]
    if kind in ("spmv", "spmm", "group"):
        n, count = case["N"] if kind == "spmm" else case["batch"], case.get("count", 1)
        wb, nnz = _matrix(case, case["M"], case["K"])
        return {"bytes": count * (wb + (case["K"] * esz + case["M"] * 4) * n), "flops": 2.0 * nnz * n * count}
    if kind in ("rnn_step", "rnn_seq"):
        H, b, T = case["H"], case["batch"], case.get("T", 1)
        total, flops = 0.0, 0.0
        for layer in range(case.get("layers", 1)):
            I = case["I"] if layer == 0 else H
            mats = [(4 * H, I + H)] if case["cell"] == "lstm" else [(3 * H, I), (3 * H, H)]
            for M, K in mats:
                wb, nnz = _matrix(case, M, K)
                total += wb + M * 4
                flops += 2.0 * nnz * b * T
                if kind == "rnn_step":
                    total += M * b * 4                       # the pre-activations, an output of the call
            # inputs, new states in the element type, the fp32 state in and out
            total += T * b * (I + H) * esz + b * H * esz + 2 * b * H * 4
        return {"bytes": total, "flops": flops}
    total, flops, osz = 0.0, 0.0, SIZE[case["out"]]
    for (ci, co, h, w, k, st, src) in _conv_layers(case):
        ho, wo = ((h + 1) // 2, (w + 1) // 2) if st == 2 else (h, w)
        wb, nnz = _matrix(case, co, ci * k * k)
        # each layer is a call of its own: reads its map, writes its map
        total += wb + co * 4 + case["batch"] * (ci * h * w * esz + co * ho * wo * osz)
        flops += 2.0 * nnz * case["batch"] * ho * wo
    return {"bytes": total, "flops": flops}


def tolerance(case):
    # Four times what the present kernels differ by from a 64-bit product of the same stored values, over a hundred cases of
    # these ranges (largest seen in brackets): sums in fp32 rel 1.5e-7, largest 8.8e-7; where results are rounded to 16
    # bits and read again, values next to a tie come out one unit apart (fp16 2^-10, bf16 2^-7 of the value).
    f16 = case["dtype"] == "f16"
    if case["kind"] == "rnn_step":
        if case["layers"] == 1:
            return {"rel": 1.2e-6, "max": 6e-6}                            # (2.6e-7, 1.5e-6)
        return {"rel": 4e-5, "max": 1e-3} if f16 else {"rel": 3e-4, "max": 8e-3}             # (fp16 9.7e-6, 2.5e-4)
    if case["kind"] == "rnn_seq":
        return {"rel": 2.4e-4, "max": 4e-3} if f16 else {"rel": 7e-4, "max": 3e-2}           # (6.0e-5, 9.7e-4; 1.7e-4, 7.8e-3)
    if case["kind"] == "conv" and case["out"] != "f32":
        return {"rel": 2e-4, "max": 4e-3} if f16 else {"rel": 4e-4, "max": 3e-2}             # (4.9e-5, 1.2e-3; 6.4e-5, 7.5e-3)
    return {"rel": 6e-7, "max": 4e-6}
