"""The work that users of this library have it do, as cases that can be prepared, run once and timed.

Four kinds of pass, each through the public entry points:

  stack    a stack of encoder layers on a batch of sentences of different lengths.  `entry` says how a program calls it:
             masked   padded tensor in, padded tensor out, one call (a serving loop; workspace and output kept)
             padded   build_offsets, then the padded stack (the offsets are wanted by the caller too)
             packed   build_offsets, pack, the packed stack, unpack (the program works on packed rows itself)
             layer    one packed layer, offsets known from before (a program with its own loop over layers)
           `fold` hands over the weight-only vectors of encoder_prepare, `shared` uses one parameter set for all layers,
           `mask` gives the batch as a 0/1 mask instead of lengths, `tanh` selects the tanh form of GELU
  mha      the variable-length attention alone, on a fused QKV buffer, with or without projection biases
  pad      the zero-padding algorithm alone around a program's own packed work: offsets, pack, unpack
  ffn      the feed-forward half of a layer from its parts: product + bias + GELU, product, add-bias + residual + LayerNorm

Lengths of a batch follow `law`: "uniform" between `lo` and `S`, "skewed" (four of five short, one of five near `S`),
"full" (every sentence has S tokens); `batch` picks the batch of that law, and the seed of the inputs the order of its
sentences.  All tensors are fp16, head size 64, weights N(0, 0.02), hidden states N(0, 1).
"""
import numpy as np
import torch

import paper_2210_03052_amd as bt

EPS = 1e-12


def listed():
    base, large = {"H": 768, "F": 3072}, {"H": 1024, "F": 4096}

    def stack(name, B, S, lo, layers, shape, entry="masked", law="uniform", fold=False, shared=False, mask=False, tanh=False):
        return {"name": name, "kind": "stack", "entry": entry, "B": B, "S": S, "lo": lo, "law": law, "batch": 1, "layers": layers,
                **shape, "fold": fold, "shared": shared, "mask": mask, "tanh": tanh}

    return [
        # a program that walks the layers itself, one full sentence: the smallest call a user makes, seven launches
        stack("layer_b1_s256", 1, 256, 256, 1, base, entry="layer", law="full"),
        # one layer on a few short sentences with offsets and padding: fixed costs only
        stack("layer_b4_s64", 4, 64, 8, 1, base),
        # interactive serving: one short request through the whole model
        stack("base_b1_s128", 1, 128, 16, 12, base),
        # serving with a small dynamic batch of requests, given as a mask
        stack("base_b8_s128", 8, 128, 26, 12, base, mask=True),
        # the ordinary inference batch (the headline configuration)
        stack("base_b16_s256", 16, 256, 51, 12, base),
        # a six-layer model whose owner prepared the fold vectors
        stack("six_layers_b16_s256_fold", 16, 256, 51, 6, base, entry="padded", fold=True),
        # one parameter set for all layers, 16 heads, tanh GELU, on packed rows
        stack("shared_b16_s256_packed", 16, 256, 51, 12, large, entry="packed", shared=True, mask=True, tanh=True),
        # long documents: attention and products of many rounds
        stack("base_b16_s1024", 16, 1024, 128, 12, base),
        # offline inference with the large shape, mostly short sentences and a few long ones: the largest call
        stack("large_b32_s512", 32, 512, 16, 24, large, law="skewed"),
        # attention alone: the ordinary batch, where it is bound by latency, and documents of the largest length allowed
        {"name": "mha_b16_s256", "kind": "mha", "B": 16, "S": 256, "lo": 1, "law": "uniform", "batch": 1, "heads": 12, "bias": False},
        {"name": "mha_b8_s4096", "kind": "mha", "B": 8, "S": 4096, "lo": 1024, "law": "uniform", "batch": 1, "heads": 16, "bias": True},
        # packing and unpacking of a large batch around other work
        {"name": "pad_b128_s512", "kind": "pad", "B": 128, "S": 512, "lo": 51, "law": "uniform", "batch": 1, "H": 768, "mask": True},
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    law = rng.choice(["uniform", "uniform", "uniform", "skewed", "full"])
    kind = rng.choice(["stack"] * 7 + ["mha"] * 2 + ["pad", "ffn"])
    if kind == "stack":
        H = rng.choice([512, 768, 768, 1024])
        S = _log(rng, 24, 1024)
        B = min(_log(rng, 1, 48), max(1, 16384 // S))
        entry = rng.choice(["masked", "masked", "padded", "packed", "layer"])
        c = {"kind": "stack", "entry": entry, "B": B, "S": S, "lo": max(1, int(S * rng.uniform(0.02, 0.6))), "law": law,
             "batch": rng.randrange(1000), "layers": 1 if entry == "layer" else rng.choice([1, 2, 4, 6, 12, 12, 24]), "H": H, "F": 4 * H,
             "fold": entry != "layer" and rng.random() < 0.25, "shared": rng.random() < 0.2,
             "mask": rng.random() < 0.5, "tanh": rng.random() < 0.3}
        while work(c)["flops"] > 2.4e12:
            c["layers"] = c["layers"] // 2
        return c
    if kind == "mha":
        S = _log(rng, 24, 4096)
        B = min(_log(rng, 1, 64), max(1, 32768 // S))
        return {"kind": "mha", "B": B, "S": S, "lo": max(1, int(S * rng.uniform(0.01, 0.6))), "law": law,
                "batch": rng.randrange(1000), "heads": rng.choice([8, 12, 12, 16]), "bias": rng.random() < 0.5}
    if kind == "pad":
        S = _log(rng, 32, 1024)
        B = min(_log(rng, 1, 256), max(1, 65536 // S))
        return {"kind": "pad", "B": B, "S": S, "lo": max(1, int(S * rng.uniform(0.02, 0.6))), "law": law,
                "batch": rng.randrange(1000), "H": rng.choice([512, 768, 768, 1024]), "mask": rng.random() < 0.5}
    H = rng.choice([512, 768, 768, 1024])
    return {"kind": "ffn", "T": _log(rng, 32, 16384), "H": H, "F": 4 * H, "tanh": rng.random() < 0.3}


# ------------------------------------------------------------------------------------------------ inputs
def _lengths(case):
    """The lengths of the batch, longest first."""
    rng = np.random.default_rng([case["batch"], case["B"], case["S"], case["lo"]])
    B, S = case["B"], case["S"]
    if case["law"] == "full":
        L = np.full(B, S)
    elif case["law"] == "skewed":  # four of five between lo and S/4, one of five in the top quarter
        long_ = int(round(0.2 * B))
        short = rng.integers(case["lo"], max(case["lo"], S // 4) + 1, B - long_)
        L = np.concatenate([short, rng.integers(max(1, 3 * S // 4), S + 1, long_)])
    else:
        L = rng.integers(case["lo"], S + 1, B)
    return np.sort(L)[::-1].astype(np.int32)


def _shuffled(case, seed):
    return np.random.default_rng(int(seed)).permutation(_lengths(case))


class _Draw:
    """Normal fp16 tensors on the GPU from a seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))

    def __call__(self, *shape, mean=0.0, std=1.0):
        return torch.empty(shape, dtype=torch.float16, device="cuda").normal_(mean, std, generator=self.g)


def _params(n, H, F):
    return {"w_qkv": n(3 * H, H, std=0.02), "b_qkv": n(3 * H, std=0.1), "w_o": n(H, H, std=0.02), "b_o": n(H, std=0.1),
            "ln0_g": n(H, mean=1.0, std=0.1), "ln0_b": n(H, std=0.1), "w_1": n(F, H, std=0.02), "b_1": n(F, std=0.1),
            "w_2": n(H, F, std=0.02), "b_2": n(H, std=0.1), "ln1_g": n(H, mean=1.0, std=0.1), "ln1_b": n(H, std=0.1),
            "heads": H // 64, "head_dim": 64, "eps": EPS}


def _batch(case, seed):
    """The batch description a program has: lengths [B] or a mask [B,S], int32, on the GPU."""
    L = _shuffled(case, seed)
    if not case["mask"]:
        return {"lengths": torch.from_numpy(L).cuda(), "S": case["S"]}
    return {"mask": torch.from_numpy((np.arange(case["S"])[None, :] < L[:, None]).astype(np.int32)).cuda()}


def prepare(case, seed):
    n = _Draw(seed)
    st = {"case": case}
    if case["kind"] == "stack":
        B, S, H, F = case["B"], case["S"], case["H"], case["F"]
        one = bt.Layer(_params(n, H, F), gelu_kind=int(case["tanh"]))
        st["layers"] = [one] + [one if case["shared"] else bt.Layer(_params(n, H, F), gelu_kind=int(case["tanh"]))
                                for _ in range(case["layers"] - 1)]
        st["fold"] = bt.encoder_prepare(st["layers"]) if case["fold"] else None
        if case["entry"] == "layer":
            L = _shuffled(case, seed)
            st["cu"], _, T, st["max_len"] = bt.build_offsets(lengths=torch.from_numpy(L).cuda(), S=S, with_max=True)
            st["x"] = n(T, H)
            st["ws"] = torch.empty(bt.layer_workspace_bytes(one, T, B, S), dtype=torch.uint8, device="cuda")
            return st
        st["batch"] = _batch(case, seed)
        st["x"] = n(B, S, H)
        st["ws"] = torch.empty(bt.layer_workspace_bytes(one, B * S, B, S), dtype=torch.uint8, device="cuda")
        st["out"] = torch.empty_like(st["x"])
    elif case["kind"] == "mha":
        L = _shuffled(case, seed)
        HD = 64 * case["heads"]
        st["cu"], _, T, st["max_len"] = bt.build_offsets(lengths=torch.from_numpy(L).cuda(), S=case["S"], with_max=True)
        st["qkv"] = n(T, 3 * HD)
        st["bias"] = [n(HD, std=0.1) for _ in range(3)] if case["bias"] else [None] * 3
    elif case["kind"] == "pad":
        st["batch"] = _batch(case, seed)
        st["x"] = n(case["B"], case["S"], case["H"])
    else:
        st["p"] = _params(n, case["H"], case["F"])
        st["x"] = n(case["T"], case["H"])
    return st


# ------------------------------------------------------------------------------------------------ one pass
def run(st):
    c = st["case"]
    if c["kind"] == "stack":
        if c["entry"] == "layer":
            return bt.encoder_layer_fwd(st["layers"][0], st["x"], st["cu"], st["max_len"], ws=st["ws"])
        if c["entry"] == "masked":
            b = st["batch"]
            out, cu, tok, T = bt.encoder_fwd_masked(st["layers"], st["x"], mask=b.get("mask"), lengths=b.get("lengths"),
                                                    out=st["out"], ws=st["ws"], fold=st["fold"])
        elif c["entry"] == "padded":
            cu, tok, T = bt.build_offsets(**st["batch"])
            out = bt.encoder_fwd_padded(st["layers"], st["x"], tok, cu, out=st["out"], ws=st["ws"], fold=st["fold"])
        else:
            cu, tok, T, longest = bt.build_offsets(**st["batch"], with_max=True)
            y = bt.encoder_fwd(st["layers"], bt.pack(st["x"], tok), cu, longest, ws=st["ws"], fold=st["fold"])
            out = bt.unpack(y, tok, c["B"], c["S"], out=st["out"])
        return {"out": out, "cu_seqlens": cu, "token_idx": tok, "tokens": T}
    if c["kind"] == "mha":
        bq, bk, bv = st["bias"]
        return bt.varlen_mha(st["qkv"], st["cu"], st["max_len"], c["heads"], bq=bq, bk=bk, bv=bv)
    if c["kind"] == "pad":
        cu, tok, T = bt.build_offsets(**st["batch"])
        packed = bt.pack(st["x"], tok)
        return {"packed": packed, "padded": bt.unpack(packed, tok, c["B"], c["S"]), "cu_seqlens": cu, "token_idx": tok}
    p = st["p"]
    g = bt.gemm_bias_act(st["x"], p["w_1"], p["b_1"], bt.ACT_GELU_TANH if c["tanh"] else bt.ACT_GELU_ERF)
    y, slices = bt.gemm_kslices(g, p["w_2"])
    if slices is None:
        y = bt.add_bias_residual_layernorm(y, p["b_2"], st["x"], p["ln1_g"], p["ln1_b"], EPS)
    else:
        y = bt.add_bias_residual_layernorm_kslices(slices, p["b_2"], st["x"], p["ln1_g"], p["ln1_b"], EPS)
    return {"hidden": g, "out": y}


def work(case):
    """Operations and bytes of one pass: every valid token's products and attention; inputs, weights and outputs once."""
    if case["kind"] == "ffn":
        T, H, F = case["T"], case["H"], case["F"]
        return {"bytes": 2.0 * (2 * H * F + 2 * T * H + T * F), "flops": 4.0 * T * H * F}
    L = _lengths(case).astype(np.float64)
    T, sq = float(L.sum()), float((L * L).sum())
    if case["kind"] == "mha":
        HD = 64 * case["heads"]
        return {"bytes": 2.0 * 4 * T * HD, "flops": 4.0 * sq * HD}
    rows, H = case["B"] * case["S"], case["H"]
    if case["kind"] == "pad":  # pack reads and writes the valid rows, unpack reads them and writes every row
        return {"bytes": 2.0 * H * (3 * T + rows) + 4.0 * (rows if case["mask"] else 0), "flops": 0.0}
    F, layers = case["F"], case["layers"]
    weights = 2.0 * (1 if case["shared"] else layers) * (4 * H * H + 2 * H * F)
    io = 2.0 * H * (2 * T if case["entry"] == "layer" else T + rows)
    return {"bytes": weights + io, "flops": layers * (2.0 * T * (4 * H * H + 2 * H * F) + 4.0 * sq * H)}


def tolerance(case):
    """fp16 storage between the steps, fp32 accumulation: a rounding is 2.8e-4 of a value, a layer has about seven in
    a row, and a stack carries them on from layer to layer.  Offsets, packing and unpacking are exact."""
    if case["kind"] == "pad":
        return "exact"
    if case["kind"] == "mha":
        return {"rel": 2e-3, "max": 0.03}
    if case["kind"] == "ffn":
        return {"rel": 2e-3, "max": 0.03}
    return {"rel": min(1e-2, 2e-3 * case["layers"] ** 0.5), "max": 0.15}
