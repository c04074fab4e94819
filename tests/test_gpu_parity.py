"""GPU parity: the HIP library, called through the C ABI, against the CPU oracle on the same
seeded inputs.  Tolerances: relative L2 over the compared outputs at most 1e-5 for fp32 storage and
2e-2 for bf16 storage, and, so that one wrong row cannot hide among many right ones, every single row
(vector along the last axis) within four times that bar, rows much smaller than the typical row being
measured on a tenth of the root-mean-square row norm."""
import numpy as np
import pytest
import torch

from oracle import classic_attention as ca
from oracle import tucker_oracle as orc
from paper_2603_30033_amd import binding as ta
from paper_2603_30033_amd import workloads as wl
from paper_2603_30033_amd.device import Layer, to_device, to_host

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-2}


def oracle_forward(w, inp, rows=None, batches=None, pos0=None):
    return orc.per_head_forward(inp["X"], wl.weights_of(inp), w.d_head, w.causal, w.rope_base,
                                pos0=w.pos0 if pos0 is None else pos0, rows=rows, batches=batches)


def run_forward(w, inp, pos0=None, with_cache=False, Lmax=None):
    with Layer(w, inp, max_positions=(w.pos0 if pos0 is None else pos0) + w.N + 8) as layer:
        X = to_device(inp["X"], w.dtype)
        Kc = Vc = None
        if with_cache:
            rt3 = w.ranks_post()[2]
            Kc = torch.zeros((w.B, Lmax, w.r3), dtype=X.dtype, device="cuda")
            Vc = torch.zeros((w.B, Lmax, rt3), dtype=X.dtype, device="cuda")
        Y = layer.forward(X, pos0=w.pos0 if pos0 is None else pos0, Kc=Kc, Vc=Vc)
        torch.cuda.synchronize()
        out = to_host(Y)
        if with_cache:
            return out, to_host(Kc), to_host(Vc)
        return out


ROW_FACTOR = 4.0


def check(y_gpu, y_ref, dtype, what=""):
    assert np.all(np.isfinite(y_gpu)), what
    err = orc.relative_l2(y_gpu, y_ref)
    assert err <= TOL[dtype], f"{what}: relative L2 {err:.3e} > {TOL[dtype]:.0e}"
    den = np.linalg.norm(np.asarray(y_ref, dtype=np.float64), axis=-1)
    rows = orc.relative_l2_rows(y_gpu, y_ref, floor=0.1 * float(np.sqrt(np.mean(den ** 2))))
    worst = float(np.max(rows)) if np.size(rows) else 0.0
    assert worst <= ROW_FACTOR * TOL[dtype], \
        f"{what}: worst row {np.unravel_index(int(np.argmax(rows)), np.shape(rows))} relative L2 {worst:.3e} > " \
        f"{ROW_FACTOR * TOL[dtype]:.0e}"
    return err


# ---- the five named workloads --------------------------------------------------------------------

def test_config1_tiny_f32_full():
    w = wl.WORKLOADS["tiny_f32"]
    inp = wl.make_inputs(w)
    check(run_forward(w, inp), oracle_forward(w, inp), w.dtype, w.name)


def test_config2_gpt2_small_scaled_full_and_full_size_sampled():
    base = wl.WORKLOADS["gpt2_small"]
    w = wl.scaled(base, B=2, N=333)                       # several tiles and a ragged tail, every row
    inp = wl.make_inputs(w)
    check(run_forward(w, inp), oracle_forward(w, inp), w.dtype, "gpt2 B=2 N=333")
    inp = wl.make_inputs(base)                            # full size, sampled rows of sampled sequences
    rows = [0, 1, 31, 32, 63, 64, 65, 127, 128, 500, 511, 512, 777, 1022, 1023]
    y = run_forward(base, inp)
    ref = oracle_forward(base, inp, rows=rows, batches=[0, 5, 7])
    check(y[[0, 5, 7]][:, rows], ref, base.dtype, "gpt2 full")


def test_config3_vit_b_scaled_full_and_full_size_sampled():
    base = wl.WORKLOADS["vit_b"]
    w = wl.scaled(base, B=3)
    inp = wl.make_inputs(w)
    check(run_forward(w, inp), oracle_forward(w, inp), w.dtype, "vit B=3")
    inp = wl.make_inputs(base)
    y = run_forward(base, inp)
    batches = [0, 100, 255]
    rows = [0, 1, 63, 64, 100, 128, 195, 196]
    ref = oracle_forward(base, inp, rows=rows, batches=batches)
    check(y[batches][:, rows], ref, base.dtype, "vit full")


def test_config4_llama_scaled_full_and_full_size_sampled():
    base = wl.WORKLOADS["llama7b_n4096"]
    w = wl.scaled(base, B=1, N=448)
    inp = wl.make_inputs(w)
    check(run_forward(w, inp), oracle_forward(w, inp), w.dtype, "llama B=1 N=448")
    inp = wl.make_inputs(base)                            # full size, every row of both sequences
    y = run_forward(base, inp)
    check(y, oracle_forward(base, inp), base.dtype, "llama full")


def test_paper_rank_shape_gpt2_8_128_64_scaled_full_and_full_size_sampled():
    base = wl.WORKLOADS["gpt2_r8_128_64"]                  # r2 != r3: query rank 128, key/value rank 64
    w = wl.scaled(base, B=2, N=300)
    inp = wl.make_inputs(w)
    check(run_forward(w, inp), oracle_forward(w, inp), w.dtype, "gpt2 [8,128,64] B=2 N=300")
    inp = wl.make_inputs(base)
    rows = [0, 1, 63, 64, 65, 511, 512, 1000, 1023]
    y = run_forward(base, inp)
    ref = oracle_forward(base, inp, rows=rows, batches=[0, 7])
    check(y[[0, 7]][:, rows], ref, base.dtype, "gpt2 [8,128,64] full")


def test_paper_rank_shape_llama1b_32_128_128_scaled_full_and_full_size_sampled():
    base = wl.WORKLOADS["llama1b_r32_128_128"]             # r1 = nH, RoPE base 5e5
    w = wl.scaled(base, B=1, N=320)
    inp = wl.make_inputs(w)
    check(run_forward(w, inp), oracle_forward(w, inp), w.dtype, "llama1b B=1 N=320")
    inp = wl.make_inputs(base)
    rows = [0, 1, 64, 1023, 1024, 2046, 2047]
    y = run_forward(base, inp)
    ref = oracle_forward(base, inp, rows=rows, batches=[0, 3])
    check(y[[0, 3]][:, rows], ref, base.dtype, "llama1b full")


def run_decode(w, inp):
    with Layer(w, inp, max_positions=int(max(inp["kv_len"])) + 1) as layer:
        x = to_device(inp["X"][:, 0], w.dtype)
        Kc, Vc = to_device(inp["Kcache"], w.dtype), to_device(inp["Vcache"], w.dtype)
        y = layer.decode(x, Kc, Vc, inp["kv_len"])
        torch.cuda.synchronize()
        return to_host(y), to_host(Kc), to_host(Vc)


def check_decode(w, inp, what):
    y, Kc, Vc = run_decode(w, inp)
    y_ref, K_ref, V_ref = orc.decode_step(inp["X"][:, 0], inp["Kcache"], inp["Vcache"], inp["kv_len"],
                                          wl.weights_of(inp), w.d_head, w.rope_base)
    check(y, y_ref, w.dtype, what)
    for b in range(w.B):
        L = int(inp["kv_len"][b])
        check(Kc[b, L - 1], K_ref[b, L - 1], w.dtype, what + " new key row")
        check(Vc[b, L - 1], V_ref[b, L - 1], w.dtype, what + " new value row")
        assert np.array_equal(Kc[b, : L - 1], inp["Kcache"][b, : L - 1])      # old rows untouched
        assert np.array_equal(Vc[b, : L - 1], inp["Vcache"][b, : L - 1])


def test_config5_decode_scaled_and_full_size():
    base = wl.WORKLOADS["decode_32k"]
    w = wl.scaled(base, B=3, kv_len=700)
    inp = wl.make_inputs(w)
    inp["kv_len"] = np.array([700, 1, 449], dtype=np.int32)                 # ragged lengths, a length-1 cache
    check_decode(w, inp, "decode B=3 ragged")
    inp = wl.make_inputs(base)
    check_decode(base, inp, "decode full")


# ---- shared key-value down-projection (one latent serves as K and V; one unrotated cache) --------

def run_decode_shared(w, inp):
    with Layer(w, inp, max_positions=int(max(inp["kv_len"])) + 1) as layer:
        x = to_device(inp["X"][:, 0], w.dtype)
        Lc = to_device(inp["Lcache"], w.dtype)
        y = layer.decode(x, Lc, None, inp["kv_len"])
        torch.cuda.synchronize()
        return to_host(y), to_host(Lc)


def check_decode_shared(w, inp, what):
    y, Lc = run_decode_shared(w, inp)
    y_ref, L_ref = orc.decode_step_shared_kv(inp["X"][:, 0], inp["Lcache"], inp["kv_len"], wl.weights_of(inp),
                                             w.d_head, w.rope_base)
    check(y, y_ref, w.dtype, what)
    for b in range(w.B):
        L = int(inp["kv_len"][b])
        check(Lc[b, L - 1], L_ref[b, L - 1], w.dtype, what + " new latent row")
        assert np.array_equal(Lc[b, : L - 1], inp["Lcache"][b, : L - 1])      # old rows untouched


# factor matrices that the projection cannot read as they lie in memory (rows or starts off 16 bytes) and a contraction that
# is one part: the new cache rows of every sequence, at its own position, and the output
@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("dtype,d,r2,r3,off", [
    ("bf16", 64, 20, 32, 0), ("bf16", 8, 6, 8, 0), ("bf16", 64, 32, 24, 1), ("f32", 64, 18, 32, 0), ("f32", 8, 8, 4, 1),
    ("f32", 40, 32, 20, 1),
])
def test_decode_of_a_narrow_model_writes_rows_at_their_positions(dtype, d, r2, r3, off, shared):
    base = wl.WORKLOADS["decode_32k_shared_kv" if shared else "decode_32k"]
    w = wl.scaled(base, d_model=d, n_heads=4, d_head=16, r1=2, r2=r2, r3=r3, rt1=2, rt2=r2, rt3=r3, B=3, kv_len=77, dtype=dtype,
                  recipe="fan_in", seed=27)
    inp = wl.make_inputs(w)
    inp["kv_len"] = np.array([77, 1, 40], dtype=np.int32)

    def moved(t):                                              # `off` elements into a larger buffer
        flat = torch.zeros(t.numel() + off, dtype=t.dtype, device="cuda")
        flat[off:] = t.flatten()
        return flat[off:].view(t.shape)

    lens = [int(n) for n in inp["kv_len"]]
    with Layer(w, inp, max_positions=78) as layer:
        layer.weights = {k: moved(v) for k, v in layer.weights.items()}
        K = to_device(inp["Lcache" if shared else "Kcache"], dtype)
        V = None if shared else to_device(inp["Vcache"], dtype)
        y = to_host(layer.decode(to_device(inp["X"][:, 0], dtype), K, V, lens))
        K, V = to_host(K), None if shared else to_host(V)
    args = (lens, wl.weights_of(inp), w.d_head, w.rope_base)
    if shared:
        y_ref, K_ref = orc.decode_step_shared_kv(inp["X"][:, 0], inp["Lcache"], *args)
    else:
        y_ref, K_ref, V_ref = orc.decode_step(inp["X"][:, 0], inp["Kcache"], inp["Vcache"], *args)
    check(y, y_ref, dtype, repr(w))
    for got, ref, old in [(K, K_ref, "Lcache")] if shared else [(K, K_ref, "Kcache"), (V, V_ref, "Vcache")]:
        for b, n in enumerate(lens):
            check(got[b, n - 1], ref[b, n - 1], dtype, f"new row of sequence {b}")
            assert np.array_equal(got[b, :n - 1], inp[old][b, :n - 1]) and np.array_equal(got[b, n:], inp[old][b, n:])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rope", [1e4, None])
def test_shared_kv_prefill_and_its_cache(dtype, rope):
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=2, N=150, dtype=dtype, rope_base=rope, seed=21, shared_kv=True, pos0=3)
    inp = wl.make_inputs(w)
    with Layer(w, inp, max_positions=w.pos0 + w.N + 8) as layer:
        X = to_device(inp["X"], w.dtype)
        Lc = torch.zeros((w.B, 200, w.r3), dtype=X.dtype, device="cuda")
        Y = layer.forward(X, pos0=w.pos0, Kc=Lc, Vc=None)
        torch.cuda.synchronize()
        check(to_host(Y), oracle_forward(w, inp), dtype, "shared-KV prefill")
        lat = inp["X"].astype(np.float64) @ inp["U3"].astype(np.float64)     # unrotated latent rows
        got = to_host(Lc)
        check(got[:, w.pos0:w.pos0 + w.N], lat, dtype, "shared-KV cache rows")
        assert not got[:, : w.pos0].any() and not got[:, w.pos0 + w.N:].any()


def test_shared_kv_llama_shape_scaled_full_and_full_size_sampled():
    base = wl.WORKLOADS["llama7b_n4096_shared_kv"]
    w = wl.scaled(base, B=1, N=320)
    inp = wl.make_inputs(w)
    check(run_forward(w, inp), oracle_forward(w, inp), w.dtype, "shared-KV llama B=1 N=320")
    inp = wl.make_inputs(base)
    y = run_forward(base, inp)
    rows = [0, 1, 64, 2047, 2048, 4094, 4095]
    ref = oracle_forward(base, inp, rows=rows, batches=[1])
    check(y[[1]][:, rows], ref, base.dtype, "shared-KV llama full")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rope", [1e4, None])
def test_shared_kv_decode_ragged(dtype, rope):
    base = wl.scaled(wl.WORKLOADS["decode_32k_shared_kv"], d_model=256, n_heads=8, d_head=32, r1=4, r2=64, r3=48,
                     B=3, kv_len=333, dtype=dtype, rope_base=rope, seed=22)
    inp = wl.make_inputs(base)
    inp["kv_len"] = np.array([333, 1, 130], dtype=np.int32)
    check_decode_shared(base, inp, "shared-KV decode ragged")


def test_shared_kv_decode_full_size():
    base = wl.WORKLOADS["decode_32k_shared_kv"]
    inp = wl.make_inputs(base)
    check_decode_shared(base, inp, "shared-KV decode full")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_shared_kv_decode_continues_a_prefill(dtype):
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=2, N=97, dtype=dtype, seed=23, shared_kv=True)
    inp = wl.make_inputs(w)
    full = oracle_forward(w, inp)                                              # causal: row N-1 = the decoded token
    with Layer(w, inp, max_positions=w.N + 1) as layer:
        X = to_device(inp["X"], w.dtype)
        Lc = torch.zeros((w.B, 128, w.r3), dtype=X.dtype, device="cuda")
        Xp = X[:, : w.N - 1].contiguous()
        layer.forward(Xp, pos0=0, Kc=Lc, Vc=None)
        y = layer.decode(X[:, w.N - 1].contiguous(), Lc, None, [w.N] * w.B)
        torch.cuda.synchronize()
        check(to_host(y), full[:, w.N - 1], dtype, "shared-KV decode after prefill")


def test_shared_kv_argument_errors():
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], N=32, shared_kv=True)
    inp = wl.make_inputs(w)
    with Layer(w, inp) as layer:
        X = to_device(inp["X"], w.dtype)
        Y = torch.empty_like(X)
        Kc = torch.zeros((w.B, 64, w.r3), dtype=X.dtype, device="cuda")
        ws = layer.workspace(ta.tucker_attn_workspace_bytes(layer.ctx, w.B, w.N))
        # a value cache has no meaning here
        assert ta.tucker_attn_forward(layer.ctx, layer.weights, X, Y, 0, Kc, Kc, ws, check=False) == -1
        x = X[:, 0].contiguous()
        wsd = layer.workspace(ta.tucker_attn_decode_workspace_bytes(layer.ctx, w.B))
        assert ta.tucker_attn_decode(layer.ctx, layer.weights, x, torch.empty_like(x), Kc, Kc, [5], wsd, check=False) == -1
    with pytest.raises(ta.TuckerAttnError):                                     # value rank must equal key rank
        ta.tucker_attn_create(d_model=64, n_heads=2, d_head=32, r1=2, r2=32, r3=32, rt3=16, shared_kv=True)


# ---- classic attention layers through the same entry point (the special cases the paper proves) --

def _selector_core(nH, dH, nG):
    """C[i, n, m] = 1 iff n = (i,l) and m = (g(i), l) (appendix lemma on D_i = A_i B_i^T)."""
    per = nH // nG
    C = np.zeros((nH, nH * dH, nG * dH), dtype=np.float32)
    for i in range(nH):
        for l in range(dH):
            C[i, i * dH + l, (i // per) * dH + l] = 1.0
    return C


def _run_weights(weights, X, d_head, causal, dtype="f32"):
    nH, r1 = weights["U1"].shape
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=X.shape[0], N=X.shape[1], d_model=X.shape[2], n_heads=nH,
                  d_head=d_head, r1=r1, r2=weights["U2"].shape[1], r3=weights["U3"].shape[1],
                  rt1=weights["Ut1"].shape[1], rt2=weights["Ut2"].shape[1], rt3=weights["Ut3"].shape[1],
                  dtype=dtype, causal=causal, rope_base=None)
    inp = {k: wl.round_to_storage(np.asarray(v, dtype=np.float32), dtype) for k, v in weights.items()}
    inp["X"] = wl.round_to_storage(X.astype(np.float32), dtype)
    return run_forward(w, inp), inp


@pytest.mark.parametrize("nG", [4, 2, 1])                       # MHA, GQA, MQA
def test_mha_gqa_mqa_through_selector_cores(nG):
    rng = np.random.default_rng(31)
    d, nH, dH, N = 64, 4, 16, 100
    g = lambda *sh: (rng.standard_normal(sh) / np.sqrt(sh[0])).astype(np.float32)
    WQ, WK, WV, WO = g(d, nH * dH), g(d, nG * dH), g(d, nG * dH), g(nH * dH, d)
    X = rng.standard_normal((2, N, d)).astype(np.float32)
    core = _selector_core(nH, dH, nG)
    eye = np.eye(nH, dtype=np.float32)
    y, inp = _run_weights(dict(C=core, U1=eye, U2=WQ, U3=WK, Ct=core, Ut1=eye, Ut2=WO.T.copy(), Ut3=WV), X, dH, True)
    for b in range(2):
        ref = ca.gqa_reference(inp["X"][b], WQ, WK, WV, WO, nH, nG, causal=True)
        check(y[b], ref, "f32", f"GQA with {nG} key-value groups")


def test_mla_through_latent_factors():
    rng = np.random.default_rng(32)
    d, nH, dH, N, dcq, dck = 64, 4, 16, 90, 40, 24
    g = lambda *sh: (rng.standard_normal(sh) / np.sqrt(sh[0])).astype(np.float32)
    WDQ, WUQ, WDKV, WUK, WDV, WUV, WO = g(d, dcq), g(dcq, nH * dH), g(d, dck), g(dck, nH * dH), g(d, dck), \
        g(dck, nH * dH), g(nH * dH, d)
    X = rng.standard_normal((1, N, d)).astype(np.float32)
    hs = lambda i: slice(i * dH, (i + 1) * dH)
    C = np.stack([WUQ[:, hs(i)] @ WUK[:, hs(i)].T for i in range(nH)]).astype(np.float32)
    Ct = np.stack([(WUV[:, hs(i)] @ WO[hs(i), :]).T for i in range(nH)]).astype(np.float32)
    eye = np.eye(nH, dtype=np.float32)
    y, inp = _run_weights(dict(C=C, U1=eye, U2=WDQ, U3=WDKV, Ct=Ct, Ut1=eye, Ut2=np.eye(d, dtype=np.float32), Ut3=WDV),
                          X, dH, True)
    # the reference consumes the up-projections; the library consumed their rounded products, so
    # compare against the oracle on exactly the library's inputs, and that against brute-force MLA
    ref_same_inputs = orc.per_head_forward(inp["X"], wl.weights_of(inp), dH, True)
    check(y, ref_same_inputs, "f32", "MLA factors")
    ref = ca.mla_reference(inp["X"][0], WDQ, WUQ, WDKV, WUK, WDV, WUV, WO, nH, causal=True)
    assert orc.relative_l2(y[0], ref) < 1e-4


# ---- edge cases ----------------------------------------------------------------------------------

@pytest.mark.parametrize("N", [1, 2, 63, 64, 65, 129])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_sequence_lengths_around_tile_edges(N, dtype):
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=2, N=N, dtype=dtype, seed=100 + N)
    inp = wl.make_inputs(w)
    check(run_forward(w, inp), oracle_forward(w, inp), dtype, f"N={N}")


@pytest.mark.parametrize("causal,rope", [(False, 1e4), (False, None), (True, None)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_mask_and_rope_switches(causal, rope, dtype):
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=2, N=150, dtype=dtype, causal=causal, rope_base=rope, seed=7)
    inp = wl.make_inputs(w)
    check(run_forward(w, inp), oracle_forward(w, inp), dtype, f"causal={causal} rope={rope}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_unequal_and_unaligned_ranks_and_odd_head_count(dtype):
    # r2 != r3, tilde ranks differ from the plain ones, none a multiple of 32, 3 heads
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=2, N=100, n_heads=3, d_model=264, d_head=88, r1=3, r2=40, r3=24,
                  rt1=2, rt2=72, rt3=56, dtype=dtype, seed=9, recipe="fan_in")
    inp = wl.make_inputs(w)
    check(run_forward(w, inp), oracle_forward(w, inp), dtype, "odd ranks")
    # wide query/output ranks, 128-wide key/value ranks
    w = wl.scaled(w, n_heads=5, r1=4, r2=160, r3=128, rt1=4, rt2=96, rt3=128, seed=10)
    inp = wl.make_inputs(w)
    check(run_forward(w, inp), oracle_forward(w, inp), dtype, "wide ranks")


def test_long_sequences():
    # 16k-token prefill (sampled rows) and a 128k-token cache in decode, both at the LLaMA-7B layer shape
    w = wl.scaled(wl.WORKLOADS["llama7b_n4096"], B=1, N=16384, seed=14)
    inp = wl.make_inputs(w)
    rows = [0, 63, 64, 4095, 8192, 12345, 16382, 16383]
    y = run_forward(w, inp)
    check(y[:, rows], oracle_forward(w, inp, rows=rows), w.dtype, "N=16384")
    wd = wl.scaled(wl.WORKLOADS["decode_32k"], B=2, kv_len=131072, seed=15)
    ind = wl.make_inputs(wd)
    ind["kv_len"] = np.array([131072, 100003], dtype=ind["kv_len"].dtype)
    ind["Kcache"][1, 100002:] = 0
    ind["Vcache"][1, 100002:] = 0
    check_decode(wd, ind, "128k-token cache")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_maximum_ranks_and_head_count(dtype):
    # every rank at the limit the library states: r1 = 64, r2 = 512, r3 = 128 (and the same after the softmax), 64 heads
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=1, N=70, n_heads=64, d_model=256, d_head=64, r1=64, r2=512, r3=128,
                  rt1=64, rt2=512, rt3=128, dtype=dtype, seed=12, recipe="fan_in")
    inp = wl.make_inputs(w)
    check(run_forward(w, inp), oracle_forward(w, inp), dtype, "maximum ranks, prefill")
    wd = wl.scaled(w, B=3, N=1, mode="decode", kv_len=150, seed=13)
    check_decode(wd, wl.make_inputs(wd), "maximum ranks, decode")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_position_offset_and_cache_outputs(dtype):
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=2, N=90, dtype=dtype, seed=11)
    inp = wl.make_inputs(w)
    y0 = run_forward(w, inp, pos0=0)
    y, Kc, Vc = run_forward(w, inp, pos0=37, with_cache=True, Lmax=160)
    ref = oracle_forward(w, inp, pos0=37)
    check(y, ref, dtype, "pos0=37")
    check(y, y0, dtype, "relative-position invariance on the GPU")
    K_ref, V_ref = orc.latent_kv(inp["X"], wl.weights_of(inp), w.rope_base, pos0=37)
    check(Kc[:, 37:127], K_ref, dtype, "cache keys")
    check(Vc[:, 37:127], V_ref, dtype, "cache values")
    assert np.all(Kc[:, :37] == 0) and np.all(Kc[:, 127:] == 0) and np.all(Vc[:, :37] == 0)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_sharp_softmax(dtype):
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=1, N=200, dtype=dtype, seed=12)
    inp = wl.make_inputs(w)
    inp["C"] = wl.round_to_storage(inp["C"] * 24.0, dtype)                   # scores of tens: near one-hot rows
    check(run_forward(w, inp), oracle_forward(w, inp), dtype, "sharp softmax")


def test_results_are_deterministic():
    w = wl.scaled(wl.WORKLOADS["gpt2_small"], B=2, N=200)
    inp = wl.make_inputs(w)
    a, b = run_forward(w, inp), run_forward(w, inp)
    assert np.array_equal(a, b)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_decode_continues_a_prefill(dtype):
    # prefill N-1 tokens with cache outputs, then decode token N-1: equals row N-1 of a causal
    # prefill of all N tokens (oracle) -- the KV-caching identity, across both entry points
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=2, N=97, dtype=dtype, seed=13)
    inp = wl.make_inputs(w)
    ref = oracle_forward(w, inp, rows=[w.N - 1])
    with Layer(w, inp, max_positions=128) as layer:
        X = to_device(inp["X"], dtype)
        Kc = torch.zeros((w.B, 128, w.r3), dtype=X.dtype, device="cuda")
        Vc = torch.zeros_like(Kc)
        layer.forward(X[:, : w.N - 1].contiguous(), Kc=Kc, Vc=Vc)
        y = layer.decode(X[:, w.N - 1].contiguous(), Kc, Vc, [w.N] * w.B)
        torch.cuda.synchronize()
        check(to_host(y), ref[:, 0], dtype, "decode after prefill")


@pytest.mark.parametrize("N", [4097, 32768])
def test_decode_continues_a_prefill_at_the_llama_shape(N):
    # the chain prefill -> cache -> decode at d = 4096, r3 = 128: N-1 tokens are prefilled with cache outputs,
    # token N-1 is decoded against that cache.  Compared with (i) the oracle's decode step on the oracle's OWN
    # cache (rotated keys and values of the same tokens) and (ii) the last row of the oracle's causal prefill.
    B = 2 if N <= 8192 else 1
    w = wl.scaled(wl.WORKLOADS["llama7b_n4096"], B=B, N=N, seed=16)
    inp = wl.make_inputs(w)
    wts = wl.weights_of(inp)
    with Layer(w, inp, max_positions=N) as layer:
        X = to_device(inp["X"], w.dtype)
        Kc = torch.zeros((B, N, w.r3), dtype=X.dtype, device="cuda")
        Vc = torch.zeros_like(Kc)
        layer.forward(X[:, : N - 1].contiguous(), Kc=Kc, Vc=Vc)
        y = layer.decode(X[:, N - 1].contiguous(), Kc, Vc, [N] * B)
        torch.cuda.synchronize()
        y, Kg, Vg = to_host(y), to_host(Kc), to_host(Vc)
    K_ref, V_ref = orc.latent_kv(inp["X"], wts, w.rope_base)
    check(Kg, K_ref, w.dtype, f"cache keys after prefill + decode, N={N}")
    check(Vg, V_ref, w.dtype, f"cache values after prefill + decode, N={N}")
    Ko, Vo = K_ref.copy(), V_ref.copy()
    Ko[:, N - 1] = 0
    Vo[:, N - 1] = 0                                       # the decode step fills the last row itself
    y_dec, _, _ = orc.decode_step(inp["X"][:, N - 1], Ko, Vo, [N] * B, wts, w.d_head, w.rope_base)
    check(y, y_dec, w.dtype, f"decode after prefill vs oracle decode on its own cache, N={N}")
    y_row = oracle_forward(w, inp, rows=[N - 1])
    check(y, y_row[:, 0], w.dtype, f"decode after prefill vs last prefill row, N={N}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_decode_edge_lengths_and_many_heads(dtype):
    base = wl.scaled(wl.WORKLOADS["decode_32k"], d_model=256, n_heads=40, d_head=32, r1=4, r2=64, r3=64,
                     dtype=dtype, B=5, kv_len=200, seed=14)
    inp = wl.make_inputs(base)
    inp["kv_len"] = np.array([200, 64, 65, 1, 129], dtype=np.int32)
    check_decode(base, inp, "decode 40 heads")


@pytest.mark.parametrize("shared,rope", [(False, 1e4), (True, 1e4), (True, None)])
@pytest.mark.parametrize("n_heads", [5, 40])
@pytest.mark.parametrize("r3", [32, 64, 128])
def test_decode_bf16_full_width_cache_rows(r3, n_heads, shared, rope):
    # bf16 caches whose rows are whole 32-channel blocks take a kernel of their own (every wave streams its own
    # keys); lengths around its 32-key blocks and 128-key rounds, a single key, and more splits than rounds
    base = wl.scaled(wl.WORKLOADS["decode_32k_shared_kv" if shared else "decode_32k"], d_model=128, n_heads=n_heads,
                     d_head=32, r1=3, r2=32, r3=r3, rt1=2, rt2=32, rt3=r3, B=7, kv_len=1100, dtype="bf16",
                     rope_base=rope, seed=31 + r3 + n_heads, recipe="fan_in")
    inp = wl.make_inputs(base)
    inp["kv_len"] = np.array([1100, 1, 31, 33, 128, 129, 517], dtype=np.int32)
    (check_decode_shared if shared else check_decode)(base, inp, "decode, full-width rows")


@pytest.mark.parametrize("shared", [False, True])
def test_decode_more_than_32_sequences(shared):
    # 70 sequences = two full passes of 32 and a ragged one, each sequence with its own cache length
    base = wl.scaled(wl.WORKLOADS["decode_32k_shared_kv" if shared else "decode_32k"], d_model=128, n_heads=6, d_head=32,
                     r1=3, r2=32, r3=48, B=70, kv_len=160, seed=17, recipe="fan_in")
    inp = wl.make_inputs(base)
    inp["kv_len"] = np.random.default_rng(5).integers(1, 161, size=70).astype(np.int32)
    (check_decode_shared if shared else check_decode)(base, inp, "decode of 70 sequences")


@pytest.mark.parametrize("seed", range(24))
def test_random_small_configurations(seed):
    """Random shapes inside the library's limits: ranks that are not multiples of the tile sizes, head
    counts that do not fill a head group, lengths around tile edges, every mode switch."""
    rng = np.random.default_rng(1000 + seed)
    dtype = ["f32", "bf16"][seed % 2]
    shared = bool(rng.integers(0, 2))
    r3 = int(rng.choice([8, 16, 24, 40, 48, 64, 72, 96, 128]))
    rt3 = r3 if shared else int(rng.choice([8, 16, 32, 56, 64, 104, 128]))
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=int(rng.integers(1, 4)), N=int(rng.integers(1, 260)),
                  d_model=int(rng.choice([64, 96, 128, 200, 256])), n_heads=int(rng.integers(1, 11)),
                  d_head=int(rng.choice([16, 32, 64])), r1=int(rng.integers(1, 5)), r2=int(rng.choice([8, 20, 32, 48, 80])),
                  r3=r3, rt1=int(rng.integers(1, 5)), rt2=int(rng.choice([8, 24, 32, 64, 100])), rt3=rt3,
                  dtype=dtype, causal=bool(rng.integers(0, 2)), rope_base=[None, 1e4, 5e5][int(rng.integers(0, 3))],
                  seed=2000 + seed, shared_kv=shared, pos0=int(rng.integers(0, 50)))
    inp = wl.make_inputs(w)
    check(run_forward(w, inp), oracle_forward(w, inp), dtype, repr(w))


@pytest.mark.parametrize("seed", range(12))
def test_random_small_decode_configurations(seed):
    rng = np.random.default_rng(3000 + seed)
    dtype = ["f32", "bf16"][seed % 2]
    shared = bool(seed % 4 >= 2)
    es = 4 if dtype == "f32" else 2
    ranks = [r for r in (8, 16, 24, 40, 48, 64, 96, 128) if (r * es) % 16 == 0]
    r3 = int(rng.choice(ranks))
    rt3 = r3 if shared else int(rng.choice(ranks))
    B = int(rng.integers(1, 6))
    kv = int(rng.integers(1, 600))
    w = wl.scaled(wl.WORKLOADS["decode_32k_shared_kv" if shared else "decode_32k"], B=B, kv_len=kv,
                  d_model=int(rng.choice([64, 128, 200])), n_heads=int(rng.integers(1, 41)), d_head=32,
                  r1=int(rng.integers(1, 5)), r2=int(rng.choice([8, 32, 48])), r3=r3, rt1=int(rng.integers(1, 5)),
                  rt2=int(rng.choice([8, 32, 64])), rt3=rt3, dtype=dtype, rope_base=[None, 1e4][int(rng.integers(0, 2))],
                  seed=4000 + seed, recipe="fan_in")
    inp = wl.make_inputs(w)
    inp["kv_len"] = rng.integers(1, kv + 1, size=B).astype(np.int32)
    if shared:
        check_decode_shared(w, inp, repr(w))
    else:
        check_decode(w, inp, repr(w))


def test_gpu_side_argument_errors():
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], N=32)
    inp = wl.make_inputs(w)
    with Layer(w, inp, max_positions=64) as layer:
        X = to_device(inp["X"], w.dtype)
        Y = torch.empty_like(X)
        ws = layer.workspace(ta.tucker_attn_workspace_bytes(layer.ctx, 1, 32))
        assert ta.tucker_attn_forward(layer.ctx, layer.weights, X, Y, 40, None, None, ws, check=False) == -1
        assert ta.tucker_attn_forward(layer.ctx, layer.weights, X, Y, 0, None, None, ws[:512], check=False) == -3
        assert ta.tucker_attn_forward(layer.ctx, layer.weights, X, Y, 0, None, None, ws, check=True) == 0
        torch.cuda.synchronize()


# ---- prepared (frozen) weights -----------------------------------------------------------------------

@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_prepared_weights_give_the_same_results_and_skip_the_preparation_kernel(dtype):
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], B=2, N=150, dtype=dtype, seed=61)
    inp = wl.make_inputs(w)
    with Layer(w, inp, max_positions=w.N + 8) as layer:
        X = to_device(inp["X"], w.dtype)
        y0 = layer.forward(X).clone()
        ta.tucker_attn_profile_enable(layer.ctx, True)
        layer.forward(X)
        plain = [n for n, _ in ta.tucker_attn_profile_read(layer.ctx)]
        layer.freeze_weights()
        y1 = layer.forward(X).clone()
        frozen = [n for n, _ in ta.tucker_attn_profile_read(layer.ctx)]
        ta.tucker_attn_profile_enable(layer.ctx, False)
        torch.cuda.synchronize()
        assert "prep_weights" in plain and "prep_weights" not in frozen
        assert torch.equal(y0, y1)
        # other weight pointers than the prepared ones are refused; after release they are accepted again
        other = dict(layer.weights, U2=layer.weights["U2"].clone())
        ws = layer.workspace(ta.tucker_attn_workspace_bytes(layer.ctx, w.B, w.N))
        assert ta.tucker_attn_forward(layer.ctx, other, X, torch.empty_like(X), 0, None, None, ws, check=False) == -1
        ta.tucker_attn_release_weights(layer.ctx)
        assert ta.tucker_attn_forward(layer.ctx, other, X, torch.empty_like(X), 0, None, None, ws, check=False) == 0
        torch.cuda.synchronize()
    check(to_host(y1), oracle_forward(w, inp), dtype, "frozen weights")


def test_prepared_weights_in_decode():
    w = wl.scaled(wl.WORKLOADS["decode_32k"], B=3, kv_len=300, d_model=256, n_heads=6, d_head=32, r1=2, r2=32, r3=64,
                  recipe="fan_in", seed=62)
    inp = wl.make_inputs(w)
    with Layer(w, inp) as layer:
        x = to_device(inp["X"][:, 0], w.dtype)
        Kc0, Vc0 = to_device(inp["Kcache"], w.dtype), to_device(inp["Vcache"], w.dtype)
        Kc1, Vc1 = Kc0.clone(), Vc0.clone()
        y0 = layer.decode(x, Kc0, Vc0, inp["kv_len"]).clone()
        layer.freeze_weights()
        y1 = layer.decode(x, Kc1, Vc1, inp["kv_len"]).clone()
        torch.cuda.synchronize()
        assert torch.equal(y0, y1) and torch.equal(Kc0, Kc1) and torch.equal(Vc0, Vc1)


def test_forward_replays_correctly_from_a_hip_graph():
    # the library only enqueues kernels on the caller's stream, so a call can be captured; every replay,
    # with fresh inputs copied into the captured buffers and eager work in between, must equal the eager result
    w = wl.scaled(wl.WORKLOADS["gpt2_small"], B=2, N=200)
    inp = wl.make_inputs(w)
    rng = np.random.default_rng(77)
    with Layer(w, inp, max_positions=w.N + 8) as layer:
        X = to_device(inp["X"], w.dtype)
        Y = torch.empty_like(X)
        ws = layer.workspace(ta.tucker_attn_workspace_bytes(layer.ctx, w.B, w.N))
        ta.tucker_attn_forward(layer.ctx, layer.weights, X, Y, 0, None, None, ws)      # first call outside the capture
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            with torch.cuda.graph(graph, stream=side):
                ta.tucker_attn_forward(layer.ctx, layer.weights, X, Y, 0, None, None, ws)
        torch.cuda.current_stream().wait_stream(side)
        for rep in range(4):
            Xn = wl.round_to_storage(rng.standard_normal(inp["X"].shape).astype(np.float32), w.dtype)
            X.copy_(to_device(Xn, w.dtype))
            Y.zero_()
            graph.replay()
            torch.cuda.synchronize()
            got = to_host(Y)
            Ye = torch.empty_like(X)
            ta.tucker_attn_forward(layer.ctx, layer.weights, X, Ye, 0, None, None, ws)  # eager, same workspace
            torch.cuda.synchronize()
            assert np.array_equal(got, to_host(Ye)), f"replay {rep}"
            check(got, orc.per_head_forward(Xn, wl.weights_of(inp), w.d_head, w.causal, w.rope_base), w.dtype, f"replay {rep}")


@pytest.mark.parametrize("shared", [False, True])
def test_decode_replays_correctly_from_a_hip_graph(shared):
    # a decode step is five kernel launches on the caller's stream (cache lengths travel by value), so a serving
    # loop can capture it; every replay, with a fresh token and eager work in between, must equal the eager result
    w = wl.scaled(wl.WORKLOADS["decode_32k_shared_kv" if shared else "decode_32k"], B=5, kv_len=700, d_model=256,
                  n_heads=12, d_head=32, r1=3, r2=64, r3=64, rt1=2, rt2=32, rt3=64, recipe="fan_in", seed=63)
    inp = wl.make_inputs(w)
    inp["kv_len"] = np.array([700, 1, 129, 512, 333], dtype=np.int32)
    lens = [int(v) for v in inp["kv_len"]]
    rng = np.random.default_rng(78)
    with Layer(w, inp, max_positions=701) as layer:
        x = to_device(inp["X"][:, 0], w.dtype)
        y = torch.empty_like(x)
        K0 = to_device(inp["Lcache" if shared else "Kcache"], w.dtype)
        V0 = None if shared else to_device(inp["Vcache"], w.dtype)
        Kc, Vc = K0.clone(), (None if shared else V0.clone())
        ws = layer.workspace(ta.tucker_attn_decode_workspace_bytes(layer.ctx, w.B))
        ta.tucker_attn_decode(layer.ctx, layer.weights, x, y, Kc, Vc, lens, ws)           # first call outside the capture
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            with torch.cuda.graph(graph, stream=side):
                ta.tucker_attn_decode(layer.ctx, layer.weights, x, y, Kc, Vc, lens, ws)
        torch.cuda.current_stream().wait_stream(side)
        for rep in range(4):
            xn = wl.round_to_storage(rng.standard_normal(inp["X"][:, 0].shape).astype(np.float32), w.dtype)
            x.copy_(to_device(xn, w.dtype))
            Kc.copy_(K0)
            if not shared:
                Vc.copy_(V0)
            y.zero_()
            graph.replay()
            torch.cuda.synchronize()
            got, gotK = to_host(y), to_host(Kc)
            Ke, Ve, ye = K0.clone(), (None if shared else V0.clone()), torch.empty_like(x)
            ta.tucker_attn_decode(layer.ctx, layer.weights, x, ye, Ke, Ve, lens, ws)      # eager, same workspace
            torch.cuda.synchronize()
            assert np.array_equal(got, to_host(ye)) and np.array_equal(gotK, to_host(Ke)), f"replay {rep}"
            if shared:
                ref, _ = orc.decode_step_shared_kv(xn, inp["Lcache"], inp["kv_len"], wl.weights_of(inp), w.d_head,
                                                   w.rope_base)
            else:
                ref, _, _ = orc.decode_step(xn, inp["Kcache"], inp["Vcache"], inp["kv_len"], wl.weights_of(inp),
                                            w.d_head, w.rope_base)
            check(got, ref, w.dtype, f"decode replay {rep}")
