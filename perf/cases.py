"""Measured workloads of the Tucker-attention library: what a program that uses it runs, over the sizes it runs it at.

Four kinds of pass, each through the public binding (`paper_2603_30033_amd.binding`, `device.from_mha_hosvd`):

  prefill    forward of B sequences of N tokens, with or without writing the latent caches
  decode     one new token per sequence against the latent cache(s), sequences of different lengths
  train      forward that saves its state, then the gradients of X and of every weight array
  convert    multi-head attention weights to Tucker weights (truncated higher-order SVD)

Layer shapes are the ones of `workloads.WORKLOADS`; `draw` varies batch, lengths, ranks, storage type and options
around them.  Inputs are made on the GPU from the seed alone, with the value recipes of `workloads.make_inputs`
(unit-variance tokens, orthonormal factors, cores of variance 1/r2).
"""
from __future__ import annotations

import math
from typing import Dict, List

import torch

from paper_2603_30033_amd import binding as ta
from paper_2603_30033_amd import device as dev

# d_model, heads, width of a head (softmax scale), and the RoPE base (0: none) and causality the layer is used with
LAYERS = {
    "tiny": (256, 4, 64, 1e4, True),
    "gpt2": (768, 12, 64, 1e4, True),
    "vit_b": (768, 12, 64, 0.0, False),
    "llama1b": (2048, 32, 64, 5e5, True),
    "llama7b": (4096, 32, 128, 1e4, True),
}
# (r1, r2, r3), used for both tensors
RANKS = {
    "tiny": [(2, 32, 32)],
    "gpt2": [(4, 64, 64), (8, 128, 64), (4, 48, 48)],
    "vit_b": [(4, 48, 48), (4, 64, 64)],
    "llama1b": [(32, 128, 128), (8, 128, 64)],
    "llama7b": [(8, 128, 128), (8, 96, 96)],
}


def _case(kind, layer, ranks, dtype="bf16", **kw):
    r1, r2, r3 = ranks
    return dict(kind=kind, layer=layer, r1=r1, r2=r2, r3=r3, dtype=dtype, **kw)


def listed() -> List[Dict]:
    return [
        # one chat on a small model: the least work a call can have, where launches and host time count
        dict(name="decode_gpt2_one", **_case("decode", "gpt2", (4, 64, 64), B=1, longest=257, ragged=False, shared=False, prepared=True)),
        # a serving batch: sequences of very different lengths, weights as the caller holds them
        dict(name="decode_llama1b_ragged", **_case("decode", "llama1b", (32, 128, 128), B=24, longest=3001, ragged=True, shared=False, prepared=False)),
        # long-context decode, two caches and one shared latent
        dict(name="decode_llama7b_32k", **_case("decode", "llama7b", (8, 128, 128), B=16, longest=32768, ragged=False, shared=False, prepared=False)),
        dict(name="decode_llama7b_32k_shared", **_case("decode", "llama7b", (8, 128, 128), B=16, longest=32768, ragged=False, shared=True, prepared=True)),
        # a chat prompt being taken in: one sequence of odd length, caches written, weights prepared once
        dict(name="prompt_llama7b_333", **_case("prefill", "llama7b", (8, 128, 128), B=1, N=333, caches=True, shared=False, prepared=True)),
        # image classification batch: many short ragged sequences, every key visible, no rotation, ranks off the tile
        dict(name="prefill_vit_b", **_case("prefill", "vit_b", (4, 48, 48), B=256, N=197, caches=False, shared=False, prepared=False)),
        # the layer forward at 4096 tokens
        dict(name="prefill_llama7b_4k", **_case("prefill", "llama7b", (8, 128, 128), B=2, N=4096, caches=False, shared=False, prepared=False)),
        # a long document taken in with one shared latent and its cache
        dict(name="prefill_llama7b_16k_shared", **_case("prefill", "llama7b", (8, 128, 128), B=1, N=16384, caches=True, shared=True, prepared=True)),
        # training steps: small layer, large layer, and the small layer in fp32 at an odd length
        dict(name="train_gpt2", **_case("train", "gpt2", (4, 64, 64), B=8, N=1024, shared=False)),
        dict(name="train_llama7b_4k", **_case("train", "llama7b", (8, 128, 128), B=2, N=4096, shared=False)),
        dict(name="train_gpt2_f32", **_case("train", "gpt2", (4, 64, 64), "f32", B=2, N=509, shared=False)),
        # a trained multi-head layer taken over into Tucker form when a model is loaded
        dict(name="convert_gpt2", **_case("convert", "gpt2", (4, 64, 64), "f32", d=768, shared=False)),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> Dict:
    kind = rng.choice(["decode", "decode", "prefill", "prefill", "prefill", "train", "train", "convert"])
    if kind == "convert":                       # layers of 4 to 12 heads of width 64
        heads = rng.randint(4, 12)
        return _case("convert", "gpt2", (4, rng.choice([32, 48, 64]), rng.choice([32, 48, 64])), "f32", d=64 * heads,
                     shared=rng.random() < 0.3)
    layer = rng.choice(["tiny", "gpt2", "vit_b", "llama1b", "llama7b"] if kind == "prefill" else ["gpt2", "llama1b", "llama7b"])
    ranks = rng.choice(RANKS[layer])
    shared = rng.random() < 0.3
    small = layer in ("tiny", "gpt2", "vit_b")
    dtype = "f32" if small and rng.random() < 0.25 else "bf16"
    if kind == "decode":
        longest = _log_int(rng, 17, 4096 if small else 32768)
        B = min(_log_int(rng, 1, 64), max(1, 16 * 32768 // longest))
        return _case("decode", layer, ranks, dtype, B=B, longest=longest, ragged=rng.random() < 0.6, shared=shared,
                     prepared=rng.random() < 0.6)
    longest = dict(tiny=512, gpt2=1024, vit_b=577, llama1b=4096, llama7b=8192)[layer]
    most = {"tiny": 8192, "gpt2": 16384, "vit_b": 65536, "llama1b": 16384, "llama7b": 8192}[layer]
    N = _log_int(rng, 16, longest)
    if kind == "train":
        N, most = max(N, 64), most // 2 if layer != "llama7b" else most
        if dtype == "f32":
            most //= 4
    B = max(1, min(256, most // N))
    B = max(1, min(B, _log_int(rng, 1, 256)))
    if kind == "train":
        return _case("train", layer, ranks, dtype, B=B, N=N, shared=shared)
    return _case("prefill", layer, ranks, dtype, B=B, N=N, caches=rng.random() < 0.4, shared=shared, prepared=rng.random() < 0.5)


# ---- inputs ---------------------------------------------------------------------------------------------------

def _torch_dtype(case):
    return dev.torch_dtype(case["dtype"])


def _orthonormal(g, rows, cols, dtype):
    """Q of a QR of a Gaussian matrix, signs fixed so that diag(R) > 0."""
    q, r = torch.linalg.qr(torch.randn(rows, cols, generator=g, device="cuda"))
    return (q * torch.sign(torch.diagonal(r))).to(dtype).contiguous()


def _normal(g, shape, std, dtype):
    return (torch.randn(*shape, generator=g, device="cuda") * std).to(dtype)


def _weights(case, g):
    d, heads, _, _, _ = LAYERS[case["layer"]]
    r1, r2, r3, dt = case["r1"], case["r2"], case["r3"], _torch_dtype(case)
    w = dict(C=_normal(g, (r1, r2, r3), r2 ** -0.5, dt), U1=_orthonormal(g, heads, r1, dt), U2=_orthonormal(g, d, r2, dt),
             U3=_orthonormal(g, d, r3, dt), Ct=_normal(g, (r1, r2, r3), r2 ** -0.5, dt), Ut1=_orthonormal(g, heads, r1, dt),
             Ut2=_orthonormal(g, d, r2, dt))
    if not case["shared"]:
        w["Ut3"] = _orthonormal(g, d, r3, dt)
    return w


class _Program:
    """What a program keeps for one layer: the context, the weights and (optionally) their prepared copies."""

    def __init__(self, case, g, max_positions, save_for_backward=False):
        d, heads, d_head, base, causal = LAYERS[case["layer"]]
        self.case = case
        self.ctx = ta.tucker_attn_create(d_model=d, n_heads=heads, d_head=d_head, r1=case["r1"], r2=case["r2"], r3=case["r3"],
                                         causal=causal, rope_base=base or None, dtype=case["dtype"], max_positions=max_positions,
                                         shared_kv=case["shared"], save_for_backward=save_for_backward)
        self.weights = _weights(case, g)
        if case.get("prepared"):
            self.prepared = torch.empty(max(ta.tucker_attn_prepared_weights_bytes(self.ctx), 256), dtype=torch.uint8, device="cuda")
            ta.tucker_attn_prepare_weights(self.ctx, self.weights, self.prepared)

    def __del__(self):
        if getattr(self, "ctx", None):
            ta.tucker_attn_destroy(self.ctx)


def _workspace(nbytes):
    return torch.empty(max(nbytes, 256), dtype=torch.uint8, device="cuda")


def prepare(case: Dict, seed: int):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if case["kind"] == "convert":
        return _prepare_convert(case, g)
    d, dt = LAYERS[case["layer"]][0], _torch_dtype(case)
    if case["kind"] == "decode":
        return _prepare_decode(case, g, d, dt)
    B, N = case["B"], case["N"]
    p = _Program(case, g, N, save_for_backward=case["kind"] == "train")
    p.X = torch.randn(B, N, d, generator=g, device="cuda").to(dt)
    p.Y = torch.empty_like(p.X)
    p.ws = _workspace(ta.tucker_attn_workspace_bytes(p.ctx, B, N))
    if case["kind"] == "train":
        p.dY = torch.randn(B, N, d, generator=g, device="cuda").to(dt)
        p.dX = torch.empty_like(p.X)
        p.grads = {"d" + k: torch.empty(v.shape, dtype=torch.float32, device="cuda") for k, v in p.weights.items()}
    else:
        p.Kc = torch.zeros(B, N, case["r3"], dtype=dt, device="cuda") if case["caches"] else None
        p.Vc = torch.zeros(B, N, case["r3"], dtype=dt, device="cuda") if case["caches"] and not case["shared"] else None
    return p


def _prepare_decode(case, g, d, dt):
    B, longest = case["B"], case["longest"]
    p = _Program(case, g, longest)
    p.x = torch.randn(B, d, generator=g, device="cuda").to(dt)
    p.y = torch.empty_like(p.x)
    # cached rows stand for rotated keys and values of unit-variance tokens, themselves unit-variance rows
    p.Kc = torch.randn(B, longest, case["r3"], generator=g, device="cuda").to(dt)
    p.Vc = None if case["shared"] else torch.randn(B, longest, case["r3"], generator=g, device="cuda").to(dt)
    # lengths depend on the case alone, so that every seed is the same amount of work
    p.lens = _lengths(case)
    p.ws = _workspace(ta.tucker_attn_decode_workspace_bytes(p.ctx, B))
    return p


def _lengths(case):
    """Cache length of every sequence: all equal, or spread evenly between one token and the longest, out of order."""
    B, longest = case["B"], case["longest"]
    if not case["ragged"] or B == 1:
        return [longest] * B
    step = next(s for s in (7, 11, 13) if B % s)
    return [1 + (longest - 1) * ((i * step) % B) // (B - 1) for i in range(B)]


class _Mha:
    pass


def _prepare_convert(case, g):
    """Stand-ins for trained projections: an orthonormal basis of the model dimension with weights j^-1/2, mixed by a
    Gaussian matrix, so that the unfoldings of the per-head products have decaying spectra as trained layers do."""
    d, dt = case["d"], _torch_dtype(case)
    s = torch.arange(1, d + 1, device="cuda", dtype=torch.float32).rsqrt()

    def one():
        mix = torch.randn(d, d, generator=g, device="cuda")
        return ((_orthonormal(g, d, d, torch.float32) * s) @ mix / s.norm()).to(dt).contiguous()

    p = _Mha()
    p.case = case
    p.WQ, p.WK, p.WV, p.WO = one(), one(), one(), one().t().contiguous()
    return p


# ---- one pass -------------------------------------------------------------------------------------------------

def run(p):
    case = p.case
    kind = case["kind"]
    if kind == "decode":
        ta.tucker_attn_decode(p.ctx, p.weights, p.x, p.y, p.Kc, p.Vc, p.lens, p.ws)
        return {"y": p.y, "K": p.Kc, "V": p.Vc}
    if kind == "prefill":
        ta.tucker_attn_forward(p.ctx, p.weights, p.X, p.Y, 0, p.Kc, p.Vc, p.ws)
        return {"Y": p.Y, "K": p.Kc, "V": p.Vc}
    if kind == "train":
        ta.tucker_attn_forward(p.ctx, p.weights, p.X, p.Y, 0, None, None, p.ws)
        ta.tucker_attn_backward(p.ctx, p.weights, p.X, p.dY, p.dX, p.grads, 0, p.ws, forward_state=True)
        return {"Y": p.Y, "dX": p.dX, **p.grads}
    ranks = (case["r1"], case["r2"], case["r3"])
    out, _ = dev.from_mha_hosvd(p.WQ, p.WK, p.WV, p.WO, case["d"] // 64, ranks, ranks, shared_kv=case["shared"])
    return out


# ---- what a pass cannot do without -------------------------------------------------------------------------------

def work(case: Dict) -> Dict:
    es = 2 if case["dtype"] == "bf16" else 4
    r1, r2, r3, vcaches = case["r1"], case["r2"], case["r3"], 1 if case["shared"] else 2
    if case["kind"] == "convert":
        # Gram matrices of the d-wide unfoldings from the head factors, four symmetric eigenproblems (reduction to
        # tridiagonal form, 4/3 d^3, and the leading r vectors back, 4 d^2 r), and the two cores
        d, heads = case["d"], case["d"] // 64
        n = 3 if case["shared"] else 4
        gram = n * (2 * d * d * 64 * heads + 2 * d * d * d)
        eig = n * (4 * d ** 3 // 3) + 2 * 4 * d * d * (r2 + r3)
        core = 2 * heads * (2 * d * 64 * (r2 + r3) + 2 * r2 * r3 * 64 + 2 * r1 * r2 * r3)
        return dict(bytes=4 * d * d * es + 2 * (r1 * r2 * r3 + heads * r1 + d * (r2 + r3)) * es, flops=gram + eig + core)
    d, heads, _, _, causal = LAYERS[case["layer"]]
    weights = 2 * (r1 * r2 * r3 + heads * r1) + d * (2 * r2 + vcaches * r3)
    if case["kind"] == "decode":
        T, pairs = case["B"], sum(_lengths(case))
        rows = pairs * r3 * vcaches
    else:
        B, N = case["B"], case["N"]
        T, pairs = B * N, B * (N * (N + 1) // 2 if causal else N * N)
        rows = 0
        if case.get("caches"):
            rows = T * r3 * vcaches
    proj = 2 * T * d * (r2 + vcaches * r3)
    mixed = min(2 * T * heads * r2 * r3, 2 * T * r1 * r2 * r3 + 2 * T * heads * r1 * r3)    # per-head query; head merge alike
    out = 2 * T * r2 * d
    dense, attn = proj + 2 * mixed + out, heads * pairs * 4 * r3
    nbytes = (weights + rows + 2 * T * d) * es
    if case["kind"] == "train":
        # the backward reads X and dY and writes dX and the fp32 gradients; each product of the forward has two gradient
        # products, the attention five products per visible pair
        return dict(bytes=nbytes + (weights + 3 * T * d) * es + weights * 4, flops=3 * dense + attn + heads * pairs * 10 * r3)
    return dict(bytes=nbytes, flops=dense + attn)


def tolerance(case: Dict) -> Dict:
    # four times what the present code measures against fp64 references on the same stored inputs, at 64 to 512 tokens
    # of these layers: bf16 rel 2.8e-3 to 6.5e-3, max 0.009 to 0.118; fp32 rel 0.7e-6 to 1.7e-6, max 2e-6 to 1.6e-5;
    # conversions (fp64 inside, rounded once to fp32) rel 2.9e-8, max 6e-8
    if case["kind"] == "convert":
        return {"rel": 1e-7, "max": 3e-7}
    if case["dtype"] == "f32":
        return {"rel": 7e-6, "max": 7e-5}
    return {"rel": 2e-2, "max": 0.5}
