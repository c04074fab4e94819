"""Sizes at which the kernels' tilings change: every tile of a dispatch rule, with remainders in the tokens, the
contraction and the heads, against the CPU oracle.  Bars as in test_gpu_parity.py (relative L2 at most 1e-5 in fp32 and
2e-2 in bf16 storage, every row within four times that)."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import tucker_oracle as orc
from paper_2603_30033_amd import binding as ta
from paper_2603_30033_amd import workloads as wl
from paper_2603_30033_amd.device import Layer, to_device, to_host
from tests.test_gpu_backward import check_all, oracle_backward, run_backward, run_case, upstream
from tests.test_gpu_parity import check, oracle_forward, run_forward

pytestmark = pytest.mark.gpu


# (dtype, sequences, tokens, model width, r2, r3, shared): the factor projection's tile at each is named in the comment
@pytest.mark.parametrize("dtype,B,N,d,r2,r3,shared", [
    ("bf16", 1, 70, 1032, 128, 96, False),      # 32 x 32, eight waves over the contraction
    ("bf16", 5, 1000, 776, 64, 64, False),      # 64 x 64
    ("bf16", 127, 130, 776, 64, 64, False),     # 96 x 128, four waves
    ("bf16", 33, 250, 1032, 128, 128, False),   # 96 x 128, eight waves
    ("bf16", 65, 250, 1032, 128, 128, True),    # 128 x 128
    ("f32", 1, 70, 264, 64, 40, False),         # 32 x 32
    ("f32", 9, 500, 264, 64, 64, False),        # 64 x 64
])
def test_projection_tiles(dtype, B, N, d, r2, r3, shared):
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=B, N=N, d_model=d, n_heads=3, d_head=32, r1=2, r2=r2, r3=r3, dtype=dtype,
                  shared_kv=shared, seed=51)
    inp = wl.make_inputs(w)
    check(run_forward(w, inp), oracle_forward(w, inp), dtype, repr(w))


# products over tokens of the backward pass: 64- and 128-wide tiles, tokens whole and split over workgroups, columns and
# rows that end inside a tile
@pytest.mark.parametrize("dtype,B,N,d,heads,r2,r3", [
    ("bf16", 1, 70, 136, 3, 48, 40),            # 64-wide, two stages, unsplit
    ("bf16", 5, 400, 136, 3, 48, 40),           # 64-wide, split
    ("bf16", 1, 130, 2056, 32, 128, 128),       # 128-wide, rows past the last whole tile
    ("f32", 3, 130, 136, 3, 48, 40),            # fp32, split
])
def test_weight_gradient_tiles(dtype, B, N, d, heads, r2, r3):
    run_case(wl.scaled(wl.WORKLOADS["tiny_f32"], B=B, N=N, d_model=d, n_heads=heads, d_head=32, r1=2, r2=r2, r3=r3,
                       dtype=dtype, seed=52))


# attention forward and backward: workgroups for few and for many (sequence, head, token) tiles, the last block of 32
# tokens partly filled and all padding
@pytest.mark.parametrize("dtype,B,N,heads,r3", [
    ("bf16", 1, 70, 3, 64), ("bf16", 2, 129, 5, 128), ("f32", 1, 97, 3, 32), ("f32", 3, 33, 4, 64),      # few
    ("bf16", 90, 130, 3, 32), ("bf16", 130, 70, 5, 64), ("f32", 90, 130, 3, 32),                         # many
])
def test_attention_workgroups(dtype, B, N, heads, r3):
    run_case(wl.scaled(wl.WORKLOADS["tiny_f32"], B=B, N=N, d_model=64, n_heads=heads, d_head=32, r1=2, r2=32, r3=r3,
                       dtype=dtype, seed=53))


# sequences of a decode step in groups of eight: a full group, one sequence more, several groups with a partial one
@pytest.mark.parametrize("B,dtype,r2,r3", [(8, "bf16", 64, 64), (9, "bf16", 160, 128), (31, "f32", 40, 32), (45, "bf16", 32, 48)])
def test_decode_sequence_groups(B, dtype, r2, r3):
    w = wl.scaled(wl.WORKLOADS["decode_32k"], B=B, kv_len=150, d_model=136, n_heads=5, d_head=32, r1=2, r2=r2, r3=r3,
                  rt1=2, rt2=r2, rt3=r3, dtype=dtype, recipe="fan_in", seed=54)
    inp = wl.make_inputs(w)
    inp["kv_len"] = np.array([1 + (37 * b) % 150 for b in range(B)], dtype=np.int32)
    with Layer(w, inp, max_positions=151) as layer:
        y = layer.decode(to_device(inp["X"][:, 0], dtype), to_device(inp["Kcache"], dtype), to_device(inp["Vcache"], dtype),
                         inp["kv_len"])
        y = to_host(y)
    ref = orc.decode_step(inp["X"][:, 0], inp["Kcache"], inp["Vcache"], inp["kv_len"], wl.weights_of(inp), w.d_head,
                          w.rope_base)[0]
    for b in range(B):
        assert orc.relative_l2(y[b], ref[b]) <= 4 * {"f32": 1e-5, "bf16": 2e-2}[dtype], b


# the same at the widths whose kernels are the tightest on registers, with enough workgroups for the large form
@pytest.mark.parametrize("dtype,r3", [("f32", 64), ("f32", 128), ("bf16", 128)])
def test_attention_workgroups_of_wide_latents(dtype, r3):
    run_case(wl.scaled(wl.WORKLOADS["tiny_f32"], B=130, N=70, d_model=64, n_heads=5, d_head=32, r1=2, r2=32, r3=r3,
                       dtype=dtype, seed=55))


# an overflown upstream gradient reaches the keys of its own block of 32 tokens and earlier ones, not later blocks
@pytest.mark.parametrize("dtype,r3", [("f32", 64), ("bf16", 32), ("bf16", 64), ("bf16", 128)])
def test_non_finite_gradients_stay_before_later_tokens(dtype, r3):
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=1, N=160, d_model=64, n_heads=3, d_head=32, r1=2, r2=32, r3=r3, dtype=dtype,
                  causal=True, seed=56)
    dY = upstream(w, 101)
    dY[0, 70] = np.inf
    dX = run_backward(w, wl.make_inputs(w), dY)["dX"]
    assert np.all(np.isfinite(dX[0, 96:])) and not np.all(np.isfinite(dX[0, 70]))


# caller's arrays that lie one element into a larger buffer: alignment to the element is all that the interface asks for
@pytest.mark.parametrize("dtype,N,d", [("f32", 70, 136), ("bf16", 70, 136), ("bf16", 1100, 1032)])
def test_arrays_that_start_on_an_element(dtype, N, d):
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=2, N=N, d_model=d, n_heads=3, d_head=32, r1=2, r2=32, r3=32, dtype=dtype,
                  seed=57)
    inp = wl.make_inputs(w)
    dY = upstream(w, 102)

    def shifted(t):
        flat = torch.zeros(t.numel() + 1, dtype=t.dtype, device=t.device)
        flat[1:] = t.flatten()
        return flat[1:].view(t.shape)

    with Layer(w, inp, max_positions=N + 8) as layer:
        X, G = to_device(inp["X"], dtype), to_device(dY, dtype)
        ctx, Y, dX = layer.ctx, shifted(torch.zeros_like(X)), shifted(torch.zeros_like(X))
        weights = {k: shifted(v) for k, v in layer.weights.items()}
        nbytes = max(ta.tucker_attn_backward_workspace_bytes(ctx, 2, N), ta.tucker_attn_decode_workspace_bytes(ctx, 2))
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        grads = {"d" + k: torch.empty(v.shape, dtype=torch.float32, device="cuda") for k, v in weights.items()}
        ta.tucker_attn_forward(ctx, weights, shifted(X), Y, workspace=ws)
        ta.tucker_attn_backward(ctx, weights, shifted(X), shifted(G), dX, grads, workspace=ws)
        y = to_host(Y)
        got = {k: to_host(v) for k, v in grads.items()}
        got["dX"] = to_host(dX)
        K, V = (torch.zeros(2, 4, 32, dtype=X.dtype, device="cuda") for _ in range(2))
        out = shifted(torch.zeros_like(X[:, 0]))                   # one token each: the first row of a causal prefill
        ta.tucker_attn_decode(ctx, weights, shifted(X[:, 0]), out, K, V, [1, 1], ws)
        out = to_host(out)
    assert orc.relative_l2(out, oracle_forward(w, inp)[:, 0]) <= {"f32": 1e-5, "bf16": 2e-2}[dtype]
    check(y, oracle_forward(w, inp), dtype, repr(w))
    check_all(got, oracle_backward(w, inp, dY), dtype, repr(w))


# attention and head merge in one launch: (sequences, tokens, heads, r2, r3, r~2); query blocks of one workgroup and of several,
# heads split over waves and not, odd head counts, a key block of one key, every width of the merged latent, values with
# and without a padding channel.  Values beyond 2^32 take the scores through the online softmax instead of the plain one.
@pytest.mark.parametrize("values", [1.0, 2.0 ** 40])
@pytest.mark.parametrize("B,N,heads,r2,r3,rt2,causal,shared", [
    (512, 1, 2, 32, 32, 32, True, False), (200, 33, 5, 40, 20, 64, True, False), (171, 96, 3, 96, 32, 96, False, False),
    (52, 290, 2, 32, 24, 40, True, True),                        # D = 32
    (256, 33, 4, 64, 48, 32, True, False), (512, 64, 3, 96, 64, 64, False, True), (150, 225, 3, 64, 48, 48, False, False),
    (100, 353, 2, 40, 64, 64, True, False), (512, 32, 8, 160, 40, 128, False, False),   # D = 64
])
def test_attention_with_the_head_merge(B, N, heads, r2, r3, rt2, causal, shared, values):
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=B, N=N, d_model=64, n_heads=heads, d_head=32, r1=2, r2=r2, r3=r3, rt1=2, rt2=rt2,
                  rt3=r3, dtype="bf16", causal=causal, shared_kv=shared, seed=58)
    inp = wl.make_inputs(w)
    if shared:
        inp["U3"] *= np.float32(values)                          # values and keys; the scores stay as they were
        inp["C"] *= np.float32(1 / values)
        inp["Ut3"] = inp["U3"]
    else:
        inp["Ut3"] *= np.float32(values)
    with Layer(w, inp) as layer:
        ta.tucker_attn_profile_enable(layer.ctx, True)
        y = to_host(layer.forward(to_device(inp["X"], w.dtype)))
        assert "attention_and_merge" in [n for n, _ in ta.tucker_attn_profile_read(layer.ctx)]
    check(y, oracle_forward(w, inp), w.dtype, repr(w))


# the same with a position offset, caches written and weights prepared before, one cache and two
@pytest.mark.parametrize("B,N,heads,r3,rt3,shared", [(200, 33, 5, 32, 20, False), (256, 40, 4, 64, 64, True), (150, 225, 3, 48, 40, False)])
def test_attention_with_the_head_merge_at_an_offset_with_caches(B, N, heads, r3, rt3, shared):
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=B, N=N, d_model=64, n_heads=heads, d_head=32, r1=2, r2=40, r3=r3, rt1=2, rt2=64,
                  rt3=rt3, dtype="bf16", causal=True, shared_kv=shared, pos0=7, seed=62)
    inp = wl.make_inputs(w)
    with Layer(w, inp, max_positions=N + 20) as layer:
        layer.freeze_weights()
        ta.tucker_attn_profile_enable(layer.ctx, True)
        K = torch.zeros(B, N + 9, r3, dtype=torch.bfloat16, device="cuda")
        V = None if shared else torch.zeros(B, N + 9, rt3, dtype=torch.bfloat16, device="cuda")
        y = to_host(layer.forward(to_device(inp["X"], w.dtype), pos0=7, Kc=K, Vc=V))
        names = [n for n, _ in ta.tucker_attn_profile_read(layer.ctx)]
        assert "attention_and_merge" in names and "prep_weights" not in names
        K, V = to_host(K), None if shared else to_host(V)
    check(y, oracle_forward(w, inp), w.dtype, repr(w))
    x = inp["X"].astype(np.float64)
    k = x @ inp["U3"].astype(np.float64)
    if not shared:
        k = np.stack([orc.rope_rotate(s, np.arange(7, 7 + N), w.rope_base) for s in k])
        check(V[:, 7:7 + N], x @ inp["Ut3"].astype(np.float64), w.dtype, "value rows")
        assert not V[:, :7].any() and not V[:, 7 + N:].any()
    check(K[:, 7:7 + N], k, w.dtype, "key rows")
    assert not K[:, :7].any() and not K[:, 7 + N:].any()


# a token without a finite value reaches the queries from its own block of 32 on, and no other sequence
@pytest.mark.parametrize("bad", [np.inf, np.nan, 3e38])
@pytest.mark.parametrize("B,N,heads,r3,rt3", [(200, 100, 5, 32, 20), (256, 70, 4, 64, 64)])
def test_attention_with_the_head_merge_of_non_finite_tokens(B, N, heads, r3, rt3, bad):
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=B, N=N, d_model=64, n_heads=heads, d_head=32, r1=2, r2=40, r3=r3, rt1=2, rt2=64,
                  rt3=rt3, dtype="bf16", causal=True, seed=63)
    inp = wl.make_inputs(w)
    ref = oracle_forward(w, inp)
    inp["X"][3, 40] = bad
    with Layer(w, inp) as layer:
        ta.tucker_attn_profile_enable(layer.ctx, True)
        y = to_host(layer.forward(to_device(inp["X"], w.dtype)))
        assert "attention_and_merge" in [n for n, _ in ta.tucker_attn_profile_read(layer.ctx)]
    assert not np.all(np.isfinite(y[3, 40]))
    check(y[3, :32], ref[3, :32], w.dtype, "queries of the block before")
    other = np.arange(B) != 3
    check(y[other], ref[other], w.dtype, "other sequences")


# queries that point away from every token's own key (scores of about -45 in powers of two, the only ones that a first token
# has) over values of 2^-100: their products lie below the smallest normal number unless the largest score is taken out first
@pytest.mark.parametrize("B,N,heads,r3,rt3", [(512, 1, 2, 32, 32), (512, 40, 3, 32, 24), (256, 33, 4, 64, 48)])
def test_attention_with_the_head_merge_of_tiny_values(B, N, heads, r3, rt3):
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=B, N=N, d_model=64, n_heads=heads, d_head=32, r1=2, r2=r3, r3=r3, rt1=2, rt2=32,
                  rt3=rt3, dtype="bf16", causal=True, seed=61)
    inp = wl.make_inputs(w)
    inp["U2"] = inp["U3"].copy()
    inp["U1"] = np.zeros_like(inp["U1"])
    inp["U1"][:, 0] = 1
    inp["C"] = np.zeros_like(inp["C"])
    inp["C"][0] = wl.round_to_storage(np.eye(r3) * (-45 * np.sqrt(32) / (1.4427 * r3)), "bf16")
    inp["Ut3"] *= np.float32(2.0 ** -100)
    with Layer(w, inp) as layer:
        ta.tucker_attn_profile_enable(layer.ctx, True)
        y = to_host(layer.forward(to_device(inp["X"], w.dtype)))
        assert "attention_and_merge" in [n for n, _ in ta.tucker_attn_profile_read(layer.ctx)]
    check(y, oracle_forward(w, inp), w.dtype, repr(w))


# projections of many tokens, one and two weight tiles of 128 and of 192 rows: whole tiles and rows past the weights, a contraction that is
# no whole stage, a last token tile that is not full
@pytest.mark.parametrize("B,N,d,r2,r3,shared", [
    (600, 33, 72, 64, 64, True), (577, 17, 136, 96, 32, False),  # 128 of 128 rows, 160 of 192
    (600, 33, 200, 64, 64, False), (519, 64, 64, 64, 64, False),  # 192 of 192
    (400, 64, 72, 128, 64, False), (512, 33, 72, 64, 128, False),  # 256 of 2 x 128, 320 of 2 x 192
])
def test_projection_of_many_tokens(B, N, d, r2, r3, shared):
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=B, N=N, d_model=d, n_heads=2, d_head=32, r1=2, r2=r2, r3=r3, rt1=2, rt2=32, rt3=r3,
                  dtype="bf16", causal=True, shared_kv=shared, seed=60)
    inp = wl.make_inputs(w)
    with Layer(w, inp) as layer:
        y = to_host(layer.forward(to_device(inp["X"], w.dtype)))
    check(y, oracle_forward(w, inp), w.dtype, repr(w))


# few workgroups: the keys of a query block dealt to two and to four waves, with a remainder and with parts that hold no visible
# key; the query blocks of a head dealt to two and to four workgroups (all gradients, no RoPE offset and an odd head count);
# parts: of the forward's keys, the query gradient's keys, the key-value gradient's queries
@pytest.mark.parametrize("dtype,B,N,heads,r3,causal,parts", [
    ("bf16", 1, 129, 3, 128, True, (2, 2, 2)), ("bf16", 1, 513, 5, 64, True, (2, 2, 2)), ("bf16", 2, 321, 4, 64, False, (2, 2, 2)),
    ("bf16", 1, 450, 3, 32, True, (4, 4, 4)), ("bf16", 2, 65, 3, 32, False, (1, 2, 4)), ("f32", 1, 65, 3, 64, True, (2, 2, 4)),
    ("f32", 1, 225, 5, 64, False, (4, 2, 4)), ("f32", 1, 97, 3, 32, True, (4, 4, 4)), ("f32", 3, 160, 3, 128, True, (2, 1, 4)),
    ("f32", 1, 96, 2, 128, False, (2, 1, 4)),
])
def test_attention_with_shared_keys(dtype, B, N, heads, r3, causal, parts):
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=B, N=N, d_model=64, n_heads=heads, d_head=32, r1=2, r2=32, r3=r3,
                  dtype=dtype, causal=causal, seed=59)
    with Layer(w, wl.make_inputs(w)) as layer:
        got = (C.c_int32 * 3)()
        ta.load_library().tucker_test_attention_parts(C.c_void_p(layer.ctx), C.c_int32(B), C.c_int32(N), got)
        assert tuple(got) == parts
    run_case(w)


# head-mixed cores: slices in batches of 4, 8 and 16 with remainders, head counts off the four of a tile, rows of a core that are no
# whole quads (prefill through the preparation launch, the last row as a decode step with the tiles in the projection's)
@pytest.mark.parametrize("dtype,heads,r1,r2,r3", [
    ("f32", 1, 1, 32, 32), ("bf16", 5, 3, 40, 30), ("f32", 7, 5, 33, 22), ("bf16", 9, 9, 48, 64), ("f32", 18, 17, 96, 32),
    ("bf16", 34, 33, 72, 40), ("bf16", 64, 64, 32, 32),
])
def test_mixed_cores(dtype, heads, r1, r2, r3):
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=2, N=40, d_model=64, n_heads=heads, d_head=32, r1=r1, r2=r2, r3=r3, dtype=dtype,
                  seed=60)
    inp = wl.make_inputs(w)
    ref = oracle_forward(w, inp)
    check(run_forward(w, inp), ref, dtype, repr(w))
    if r3 % 8 == 0:                                              # whole 16-byte chunks: what a decode step takes
        with Layer(w, inp) as layer:
            X = to_device(inp["X"], dtype)
            K, V = (torch.zeros(2, 40, r3, dtype=X.dtype, device="cuda") for _ in range(2))
            ws = torch.empty(ta.tucker_attn_workspace_bytes(layer.ctx, 2, 39), dtype=torch.uint8, device="cuda")
            head = X[:, :39].contiguous()
            ta.tucker_attn_forward(layer.ctx, layer.weights, head, torch.empty_like(head), 0, K, V, ws)
            y = to_host(layer.decode(X[:, 39].contiguous(), K, V, [40, 40]))
        check(y, ref[:, 39], dtype, repr(w))
