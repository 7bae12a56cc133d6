"""The fp32 matrix kernels at the edges of their tiles (16 query rows x 16 keys, head dimensions padded
to 64, 128 or 256, keys dealt out over four waves and over splits) against the double-precision
oracles, and the one thing a padded tile must not do: let a key reach a row that does not see it."""
import math

import numpy as np
import pytest
import torch

from parity import F32_MAX_REL, host, max_rel, oracle_decode, oracle_prefill

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def plx():
    from paper_2605_29157_amd import binding

    binding.load_library()
    return binding


@pytest.fixture(scope="module")
def synth():
    from paper_2605_29157_amd import synth as s

    return s


@pytest.mark.parametrize("T,Tkv,d,G", [(1, 1, 4, 1), (15, 15, 60, 2), (16, 16, 64, 1), (17, 17, 68, 2), (16, 79, 128, 4),
                                       (33, 64, 132, 1), (65, 65, 256, 2), (130, 131, 252, 1), (200, 200, 96, 2)])
def test_prefill_edges(plx, synth, oracle, T, Tkv, d, G):
    y = synth.prefill_inputs(2, 2 * G, 2, Tkv, d, seed=41 + T, dtype=torch.float32, device=DEV)
    y["q"], y["r"] = y["q"][:, :, Tkv - T:], y["r"][:, :, Tkv - T:]  # strided rows
    for causal, use_r in ((True, True), (False, True), (True, False)):
        got = plx.parallax_prefill(y["q"], y["r"] if use_r else None, y["k"], y["v"], y["scale"], causal=causal,
                                   use_r=use_r)
        assert max_rel(host(got), oracle_prefill(oracle, y, causal=causal, use_r=use_r)) <= F32_MAX_REL


@pytest.mark.parametrize("L,d,Hq,Hkv,Tq,S", [(1, 64, 2, 2, 1, 0), (2047, 64, 16, 8, 1, 0), (1100, 128, 8, 1, 3, 0),
                                             (700, 256, 4, 2, 1, 5), (130, 36, 6, 2, 1, 128), (3000, 68, 20, 1, 2, 0)])
def test_decode_edges_split_and_unsplit(plx, synth, oracle, L, d, Hq, Hkv, Tq, S):
    x = synth.decode_inputs(3, Hq, Hkv, L, d, seed=17 + L, dtype=torch.float32, device=DEV)
    lens = [L, max(L // 3, Tq), 0]
    x["seq_lens"] = torch.tensor(lens, dtype=torch.int32, device=DEV)
    if Tq > 1:
        more = synth.prefill_inputs(3, Hq, Hkv, Tq, d, seed=18, dtype=torch.float32, device=DEV)
        x["q"], x["r"] = more["q"], more["r"]
    outs = [plx.parallax_decode(x["q"], x["r"], x["k"], x["v"], x["scale"], seq_lens=x["seq_lens"], num_splits=s)
            for s in (S, 1)]
    for b, n in enumerate(lens):
        for out in outs:
            if n == 0:
                assert float(out[b].abs().max()) == 0.0
                continue
            q, r = (host(x[t][b:b + 1]).reshape(1, Hq, Tq, d) for t in "qr")
            ref = oracle.forward(q, r, host(x["k"][b:b + 1, :, :n]), host(x["v"][b:b + 1, :, :n]), x["scale"], causal=Tq > 1)
            assert max_rel(host(out[b]).reshape(ref.shape), ref) <= F32_MAX_REL
    # a workspace that is too small for the split count: the call runs unsplit
    few = plx.parallax_decode(x["q"], x["r"], x["k"], x["v"], x["scale"], seq_lens=x["seq_lens"], num_splits=S,
                              workspace=torch.empty(4, dtype=torch.float32, device=DEV))
    assert torch.equal(few, outs[1])


def test_a_split_of_nan_keys_is_not_dropped(plx, synth):
    """The last of four splits (keys 1536 on) holds NaN keys only: the row has no result (zeros, as unsplit), not the
    result of the other splits."""
    x = synth.decode_inputs(2, 4, 2, 2000, 64, seed=31, dtype=torch.float32, device=DEV)
    x["k"][1, :, 1536:] = math.nan
    outs = [plx.parallax_decode(x["q"], x["r"], x["k"], x["v"], x["scale"], num_splits=s) for s in (1, 4)]
    for out in outs:
        assert float(out[0].abs().max()) > 0.0 and float(out[1].abs().max()) == 0.0


@pytest.mark.parametrize("bad", [math.nan, math.inf])
@pytest.mark.parametrize("T,d,window", [(50, 64, 0), (40, 128, 9), (37, 256, 0)])
def test_a_row_ignores_what_it_does_not_see(plx, synth, T, d, window, bad):
    """Key `at` holds inf / NaN: rows that do not see it come out as without it, in the forward and in
    the row gradients; in the key gradients the same for a row that does not see a key."""
    y = synth.prefill_inputs(1, 2, 1, T, d, seed=77, dtype=torch.float32, device=DEV)
    d_o = synth.prefill_inputs(1, 2, 1, T, d, seed=78, dtype=torch.float32, device=DEV)["q"]
    at = T // 2 + 1

    def step(z, g):
        o, vbar, st = plx.parallax_prefill(z["q"], z["r"], z["k"], z["v"], z["scale"], save_for_backward=True, window=window)
        return [o, *plx.parallax_prefill_backward(z["q"], z["r"], z["k"], z["v"], o, vbar, st, g, z["scale"], window=window)]

    clean = step(y, d_o)
    for name in "kv":
        z = {n: (t.clone() if torch.is_tensor(t) else t) for n, t in y.items()}
        z[name][:, :, at, 3] = bad
        got = step(z, d_o)
        blind = [i for i in range(T) if i < at or (window and i >= at + window)]
        for a, b in zip(got[:3], clean[:3]):  # o, dq, dr
            np.testing.assert_allclose(host(a)[:, :, blind], host(b)[:, :, blind], rtol=1e-5, atol=1e-5)
    g = d_o.clone()
    g[:, :, at, 3] = bad
    got = step(y, g)
    blind = [j for j in range(T) if j > at or (window and j <= at - window)]
    for a, b in zip(got[3:], clean[3:]):  # dk, dv
        np.testing.assert_allclose(host(a)[:, :, blind], host(b)[:, :, blind], rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("bad", [math.nan, math.inf, -math.inf])
@pytest.mark.parametrize("T,d", [(50, 64), (37, 100), (37, 128), (40, 200), (37, 256)])
@pytest.mark.parametrize("use_r", [True, False])
@pytest.mark.parametrize("low", [False, True])
def test_a_row_takes_what_it_sees(plx, synth, T, d, use_r, bad, low):
    """A value that is not finite, in a block of keys that some rows see only in part: it is in the
    outputs of the rows that see the key, in its own dimension and no other, also where the weight of
    the key is zero (low: its score lies hundreds of binades down), and in no other row."""
    y = synth.prefill_inputs(1, 2, 1, T, d, seed=79, dtype=torch.float32, device=DEV)
    at, dim = T // 2 + 1, 3
    if low:
        y["q"] = y["q"].abs() + 1.0
        y["k"][:, :, at] = -100.0
        y["r"] = 0.0 * y["r"]  # (keeps the key's finite dimensions comparable)
    args = (y["q"], y["r"] if use_r else None, y["k"])
    clean = plx.parallax_prefill(*args, y["v"], y["scale"], use_r=use_r)
    v = y["v"].clone()
    v[:, :, at, dim] = bad
    got = plx.parallax_prefill(*args, v, y["scale"], use_r=use_r)
    assert not torch.isfinite(got[:, :, at:, dim]).any()
    if math.isnan(bad) or low:
        assert torch.isnan(got[:, :, at:, dim]).all()
    elif not use_r:
        assert (got[:, :, at:, dim] == bad).all()
    rest = torch.ones_like(got, dtype=torch.bool)
    rest[:, :, at:, dim] = False
    assert torch.equal(got[rest], clean[rest])
