"""Prefill with the keys of a row block split over workgroups, against the oracle and against the
whole launch (parallax_prefill through the C ABI), at the shapes where a range can go wrong: ranges that
start on the diagonal (rows that see nothing of them), a last range of one key, one range only for the
short row blocks."""
import ctypes

import numpy as np
import pytest
import torch

from parity import BF16_REL_L2, host, oracle_prefill, rel_l2

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


def _inputs(synth, B, Hq, Hkv, T, Tkv, d, seed):
    y = synth.prefill_inputs(B, Hq, Hkv, Tkv, d, seed=seed, device=DEV, k_offset_sigma=0.5)
    y["q"], y["r"] = y["q"][:, :, Tkv - T:].contiguous(), y["r"][:, :, Tkv - T:].contiguous()
    return y


def _whole(plx, y, causal=True, use_r=True, stats=False):
    out = torch.empty_like(y["q"])
    a = plx.prefill_args(y["q"], y["r"], y["k"], y["v"], out, y["scale"], causal, use_r)
    vbar = torch.empty_like(out)
    st = torch.empty(y["q"].shape[:3] + (2,), dtype=torch.float32, device=DEV)
    if stats:
        a.vbar, a.row_stats = vbar.data_ptr(), st.data_ptr()
    lib = plx.load_library()
    need = lib.parallax_prefill_workspace_bytes(ctypes.byref(a))
    assert (lib.parallax_prefill_form(ctypes.byref(a), need) >= 256) == (need > 0)  # scratch is asked for by calls that are split
    assert lib.parallax_prefill(ctypes.byref(a), None) == 0
    return (out, vbar, st) if stats else out, need


# (B, Hq, Hkv, T, Tkv, d): heads * row blocks leave most of the chip idle
SHAPES = [(1, 1, 1, 1500, 1501, 128), (1, 2, 1, 300, 1281, 128), (1, 2, 2, 130, 5000, 128), (2, 4, 4, 17, 3001, 128),
          (1, 2, 2, 512, 1600, 128), (1, 1, 1, 1500, 1500, 64), (1, 2, 1, 700, 2625, 64), (1, 4, 4, 300, 2049, 64)]


@pytest.mark.parametrize("B,Hq,Hkv,T,Tkv,d", SHAPES)
def test_the_records_are_written(plx, synth, B, Hq, Hkv, T, Tkv, d):
    """A call that says it is split goes through its scratch: every row's record is there afterwards; one that is
    given too little leaves it alone."""
    y = _inputs(synth, B, Hq, Hkv, T, Tkv, d, 4050 + T)
    whole, need = _whole(plx, y)
    out, lib = torch.empty_like(whole), plx.load_library()
    a = plx.prefill_args(y["q"], y["r"], y["k"], y["v"], out, y["scale"], True, True)
    form = lib.parallax_prefill_form(ctypes.byref(a), need)
    ws = torch.full((need // 4,), -7.25, dtype=torch.float32, device=DEV)
    assert lib.parallax_prefill_split(ctypes.byref(a), ws.data_ptr(), need - 4, None) == 0
    assert bool((ws == -7.25).all()) and torch.equal(out, whole)
    assert lib.parallax_prefill_split(ctypes.byref(a), ws.data_ptr(), need, None) == 0
    torch.cuda.synchronize()
    assert torch.equal(out, plx.parallax_prefill(y["q"], y["r"], y["k"], y["v"], y["scale"]))
    # records [B * Hq][items][4 x 32 rows][64 d + 160]: those of row blocks with more than one range
    rec = ws.reshape(B * Hq, -1, 4, 64 * d + 160)
    item, nrb = 0, -(-T // 128)
    for rb in range(nrb - 1, -1, -1):
        tiles = -(-min(Tkv, (rb + 1) * 128 + Tkv - T) // 64)
        count = -(-tiles // (form // 256))
        waves = -(-min(128, T - rb * 128) // 32)
        written = rec[:, item:item + count] != -7.25
        assert bool(written[:, :, :waves, :64 * d + 96].all()) == (count > 1)
        assert not bool(written[:, :, waves:].any()) and (count > 1 or not bool(written.any()))
        item += count
    assert item == rec.shape[1]


@pytest.mark.parametrize("B,Hq,Hkv,T,Tkv,d", SHAPES)
@pytest.mark.parametrize("causal,use_r", [(True, True), (False, True), (True, False)])
def test_split_prefill(plx, synth, oracle, B, Hq, Hkv, T, Tkv, d, causal, use_r):
    y = _inputs(synth, B, Hq, Hkv, T, Tkv, d, 4100 + T)
    whole, need = _whole(plx, y, causal, use_r)
    assert need > 0
    got = plx.parallax_prefill(y["q"], y["r"], y["k"], y["v"], y["scale"], causal=causal, use_r=use_r)
    torch.cuda.synchronize()
    ref = oracle_prefill(oracle, y, causal=causal, use_r=use_r)
    assert rel_l2(host(got), ref) <= BF16_REL_L2
    # (both within the bf16 bound of the oracle, and of each other)
    assert rel_l2(host(got), host(whole).astype(np.float64)) <= BF16_REL_L2
    if causal and T == Tkv:
        assert torch.equal(got[:, :, 0], y["v"][:, :, 0].repeat_interleave(Hq // Hkv, 1))  # one key: v_0 exactly


@pytest.mark.parametrize("B,Hq,Hkv,T,Tkv,d", SHAPES)
@pytest.mark.parametrize("causal", [True, False])
def test_split_prefill_rounds_like_the_whole_launch(plx, synth, B, Hq, Hkv, T, Tkv, d, causal):
    """All ranges share the reference of the whole launch, so P is rounded to the same bf16 values and what
    is left is the order of fp32 sums (and, in a range's last step, whether a sum takes P before or after
    its rounding): outputs a rounding step of bf16 apart here and there. Ranges with references of
    their own differ by 2.9e-3."""
    y = _inputs(synth, B, Hq, Hkv, T, Tkv, d, 4250 + T)
    whole, need = _whole(plx, y, causal)
    assert need > 0
    got = plx.parallax_prefill(y["q"], y["r"], y["k"], y["v"], y["scale"], causal=causal)
    e = rel_l2(host(got), host(whole).astype(np.float64))
    print("rel", e)
    assert e <= 1e-3


@pytest.mark.parametrize("B,Hq,Hkv,T,Tkv,d", SHAPES)
def test_split_prefill_row_cache(plx, synth, B, Hq, Hkv, T, Tkv, d):
    y = _inputs(synth, B, Hq, Hkv, T, Tkv, d, 4200 + T)
    (o, vbar, st), need = _whole(plx, y, stats=True)
    assert need > 0
    go, gv, gs = plx.parallax_prefill(y["q"], y["r"], y["k"], y["v"], y["scale"], save_for_backward=True)
    torch.cuda.synchronize()
    assert rel_l2(host(go), host(o).astype(np.float64)) <= BF16_REL_L2
    assert rel_l2(host(gv), host(vbar).astype(np.float64)) <= BF16_REL_L2
    # fp32 sums of the unrounded P1, P2 either way
    np.testing.assert_allclose(host(gs)[..., 0], host(st)[..., 0], rtol=0, atol=2e-4)
    np.testing.assert_allclose(host(gs)[..., 1], host(st)[..., 1], rtol=1e-3, atol=2e-3)


def test_logits_that_grow_along_the_sequence(plx, synth, oracle):
    """References of the ranges hundreds of binades apart: the early ranges merge away to nothing, and a
    range whose own reference does not hold takes the online update."""
    y = _inputs(synth, 1, 2, 2, 200, 3000, 128, 4300)
    ramp = torch.linspace(0.1, 30.0, 3000, device=DEV)[None, None, :, None]
    y["q"] = y["q"].abs().to(torch.bfloat16)
    y["k"] = (ramp * torch.ones_like(y["k"])).to(torch.bfloat16)
    y["r"] = (0.01 * y["r"]).to(torch.bfloat16)
    _, need = _whole(plx, y)
    assert need > 0
    got = plx.parallax_prefill(y["q"], y["r"], y["k"], y["v"], y["scale"])
    assert rel_l2(host(got), oracle_prefill(oracle, y)) <= BF16_REL_L2


@pytest.mark.parametrize("d,high", [(128, 7.75), (64, 10.9375)])  # 126.5 and 126.2 binades above the other keys
@pytest.mark.parametrize("where", ["late_then_first", "late_everywhere"])
def test_ranges_whose_sums_come_close_to_the_end_of_fp32(plx, synth, oracle, d, high, where):
    """A range keeps its reference, the first 32 keys, as long as its sums are finite. Late in the first range
    and first in the second: two sums close to the end of fp32 (with references of their own: the
    ranges weigh the same, at references 126 binades apart). Late in every range: each sum is finite,
    their total is not."""
    T, Tkv = 32, 4096
    y = _inputs(synth, 1, 2, 2, T, Tkv, d, 4500)
    _, need = _whole(plx, y)
    ranges = need // (2 * 4 * (64 * d + 160) * 4)
    tiles = -(-(Tkv // 64) // ranges)
    assert ranges >= 4 and tiles >= 2
    first = [64 * tiles * i for i in range(ranges)]
    at = [40, first[1]] if where == "late_then_first" else [x + 40 for x in first]
    y["q"] = torch.ones_like(y["q"])
    y["k"] = torch.zeros_like(y["k"])
    y["k"][:, :, at] = high
    y["r"], y["v"] = (0.002 * y["r"]).to(torch.bfloat16), (0.2 * y["v"]).to(torch.bfloat16)
    (whole, vbar, st), _ = _whole(plx, y, stats=True)
    got, gv, gs = plx.parallax_prefill(y["q"], y["r"], y["k"], y["v"], y["scale"], save_for_backward=True)
    plain = plx.parallax_prefill(y["q"], y["r"], y["k"], y["v"], y["scale"])
    ref = oracle_prefill(oracle, y)
    assert rel_l2(host(whole), ref) <= BF16_REL_L2
    assert rel_l2(host(got), ref) <= BF16_REL_L2 and rel_l2(host(plain), ref) <= BF16_REL_L2
    assert rel_l2(host(gv), host(vbar).astype(np.float64)) <= BF16_REL_L2
    np.testing.assert_allclose(host(gs), host(st), rtol=1e-5, atol=2e-3)


def test_small_workspace_and_full_chip_run_whole(plx, synth):
    y = _inputs(synth, 1, 2, 2, 130, 5000, 128, 4400)
    whole, need = _whole(plx, y)
    out = torch.empty_like(whole)
    a = plx.prefill_args(y["q"], y["r"], y["k"], y["v"], out, y["scale"], True, True)
    ws = torch.empty(need // 4, dtype=torch.float32, device=DEV)
    lib = plx.load_library()
    assert lib.parallax_prefill_split(ctypes.byref(a), ws.data_ptr(), need - 4, None) == 0
    torch.cuda.synchronize()
    assert torch.equal(out, whole)
    assert lib.parallax_prefill_split(ctypes.byref(a), ws.data_ptr() + 4, need, None) == plx.PLX_ERR_WORKSPACE
    y = _inputs(synth, 4, 16, 8, 1024, 1024, 128, 4401)
    assert _whole(plx, y)[1] == 0
