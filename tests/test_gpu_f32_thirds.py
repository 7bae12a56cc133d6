"""Large fp32 prefill launches at d = 64 (bf16 thirds) at the edges of their tiles (32 columns x 32 keys, two tiles at a
time): against the double-precision oracle, and against the fp32 matrix kernels that a launch of one key head runs."""
import ctypes
import math

import numpy as np
import pytest
import torch

from parity import host, rel_l2

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# Three thirds hold 24 bits (from 2^-110 on). Of the products the three smallest are left out: a first third is cut off, so the
# second can reach 2^-7 of its value and the third 2^-16, and second by third, twice, 2^-22 of a product at most (over random
# values 3.8 * 2^-24 has been seen, 0.4 * 2^-24 rms). Those and about 400 roundings at 2^-24, all of random sign, make 20 * 2^-24 =
# 1.2e-6 of a sum.
REL = 1.2e-6


@pytest.fixture(scope="module")
def plx():
    from paper_2605_29157_amd import binding

    binding.load_library()
    return binding


def _inputs(B, Hq, Hkv, T, Tkv, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    shapes = dict(q=(B, Hq, T, 64), r=(B, Hq, T, 64), k=(B, Hkv, Tkv, 64), v=(B, Hkv, Tkv, 64), g=(B, Hq, T, 64))
    return {n: torch.randn(s, generator=gen, device=DEV) for n, s in shapes.items()}


def _step(plx, x, causal=True, window=0):
    o, vbar, st = plx.parallax_prefill(x["q"], x["r"], x["k"], x["v"], 0.125, causal=causal, window=window, save_for_backward=True)
    return [o, *plx.parallax_prefill_backward(x["q"], x["r"], x["k"], x["v"], o, vbar, st, x["g"], 0.125, causal=causal,
                                              window=window)]


def _one_head(x, b, hk):
    G = x["q"].shape[1] // x["k"].shape[1]
    heads = lambda n: slice(hk, hk + 1) if n in "kv" else slice(hk * G, hk * G + G)
    return {n: torch.empty_like(t[b:b + 1, heads(n)], memory_format=torch.contiguous_format).copy_(t[b:b + 1, heads(n)]) for n, t in x.items()}


def _head_of(outs, b, hk, G):
    return [t[b:b + 1, hk:hk + 1] if n > 2 else t[b:b + 1, hk * G:hk * G + G] for n, t in enumerate(outs)]


def _forms(plx, x, causal=True, window=0):
    """32 where a launch runs in thirds: the forward, the backward's pass over the rows, and that over the keys."""
    lib = plx.load_library()
    a = plx.prefill_args(x["q"], x["r"], x["k"], x["v"], torch.empty_like(x["q"]), 0.125, causal, True, window)
    B, Hq, T, _ = x["q"].shape
    stats, ws = torch.empty(B, Hq, T, 2, device=DEV), torch.empty(B * Hq * T * 4, device=DEV)
    b = plx.prefill_bwd_args(x["q"], x["r"], x["k"], x["v"], x["q"], x["q"], stats, x["g"], x["q"], x["q"], x["k"], x["v"], 0.125, causal,
                             ws, window)
    back = lib.parallax_prefill_backward_form(ctypes.byref(b))
    return lib.parallax_prefill_form(ctypes.byref(a), 0), back // 256, back % 256


@pytest.mark.parametrize("B,Hq,Hkv,T,Tkv,causal,window", [
    # (several query heads to a key head: items of a pass over the keys that cross from one head to the next two at a time, odd
    # numbers of them a head and in all, windows, more keys than rows)
    (4, 64, 32, 129, 223, True, 0), (2, 96, 32, 257, 257, True, 0), (4, 64, 32, 225, 300, True, 130), (3, 96, 32, 161, 225, False, 0),
    (8, 16, 16, 128, 128, True, 0), (4, 32, 32, 257, 257, True, 0), (4, 32, 16, 161, 225, True, 0), (4, 32, 32, 159, 223, True, 0),
    (5, 26, 26, 160, 161, False, 0), (4, 32, 32, 190, 128, False, 0), (4, 32, 32, 230, 230, True, 96), (4, 32, 32, 193, 320, True, 101)])
def test_thirds_at_the_edges(plx, B, Hq, Hkv, T, Tkv, causal, window):
    from oracle import parallax_backward

    x = _inputs(B, Hq, Hkv, T, Tkv, seed=T + Tkv)
    forms = _forms(plx, x, causal, window)
    assert forms == (32, 32, 32 if Hkv * B * -(-Tkv // 32) >= 512 else 0)
    outs, G = _step(plx, x, causal, window), Hq // Hkv
    for b, hk in ((0, 0), (B - 1, Hkv - 1)):
        one = _one_head(x, b, hk)
        few = _step(plx, one, causal, window)
        args = [host(one[n]) for n in "qrkv"]
        want = [parallax_backward.forward_with_cache(*args, 0.125, causal=causal, window=window)[0],
                *parallax_backward.backward(*args, host(one["g"]), 0.125, causal=causal, window=window)]
        for name, got, fp32, ref in zip(("o", "dq", "dr", "dk", "dv"), _head_of(outs, b, hk, G), few, want):
            assert rel_l2(host(got), ref) <= REL, (name, rel_l2(host(got), ref))
            if name in ("o", "dq", "dr") or forms[2]:
                assert not torch.equal(got, fp32), (name, "the launch did not run the kernels under test")
                assert rel_l2(host(got), ref) <= rel_l2(host(fp32), ref), name


@pytest.mark.parametrize("B,Hq,Hkv,T,Tkv,causal,window", [
    (16, 8, 8, 129, 129, True, 0), (16, 8, 8, 176, 176, True, 0), (16, 16, 16, 208, 208, True, 0), (8, 16, 16, 144, 144, False, 0),
    (8, 16, 16, 128, 140, True, 0), (4, 8, 8, 1024, 1024, True, 1), (4, 8, 8, 1024, 1024, True, 64)])
def test_launches_of_half_empty_tiles_stay_on_the_fp32_instruction(plx, B, Hq, Hkv, T, Tkv, causal, window):
    """Just above a pair of tiles, few keys to a row, or a narrow window: up to half as long again in thirds. Bits of the
    kernels that a launch of one head runs."""
    x = _inputs(B, Hq, Hkv, T, Tkv, seed=T)
    assert _forms(plx, x, causal, window) == (0, 0, 0)
    few = _step(plx, _one_head(x, B - 1, 3), causal, window)
    for name, got, want in zip(("o", "dq", "dr", "dk", "dv"), _head_of(_step(plx, x, causal, window), B - 1, 3, 1), few):
        assert torch.equal(got, want), name


def test_forward_without_probe_and_with_strided_rows(plx):
    x = _inputs(4, 32, 32, 300, 300, seed=5)
    y = {n: t[:, :, 40:] if n in "qr" else t for n, t in x.items()}
    assert _forms(plx, _inputs(4, 32, 32, 260, 300, seed=5)) == (32, 32, 32)  # (of the same shape, dense)
    for use_r in (True, False):
        got = plx.parallax_prefill(y["q"], y["r"] if use_r else None, y["k"], y["v"], 0.125, use_r=use_r)
        one = {n: t[3:, 31:] for n, t in y.items()}
        few = plx.parallax_prefill(one["q"], one["r"] if use_r else None, one["k"], one["v"], 0.125, use_r=use_r)
        assert not torch.equal(got[3:, 31:], few)
        assert rel_l2(host(got[3:, 31:]), host(few).astype(np.float64)) <= REL


@pytest.mark.parametrize("scales", [dict(v=1e-30), dict(v=1e35, g=1e-30), dict(g=1e-28), dict(k=1e-18, q=1e18), dict(v=3e-36),
                                    dict(g=1e-36)])
def test_small_and_large_values(plx, scales):
    """Powers of ten that leave thirds below the smallest number, or near the largest."""
    x = _inputs(4, 32, 32, 226, 226, seed=9)
    assert _forms(plx, x) == (32, 32, 32)
    for n, f in scales.items():
        x[n] *= f
    outs, few = _step(plx, x), _step(plx, _one_head(x, 2, 7))
    for name, got, ref in zip(("o", "dq", "dr", "dk", "dv"), _head_of(outs, 2, 7, 1), few):
        a, b = host(got).astype(np.float64), host(ref).astype(np.float64)
        assert np.isfinite(a).all() and np.isfinite(b).all(), name
        size = np.abs(b).max() or 1.0
        assert rel_l2(a / size, b / size) <= 2 * REL, name


def _times(x, factor, *names):
    for n in names:
        x[n] *= factor


# What is scaled by tiny and huge factors, and which parts of which results are looked at (those that do not underflow).
# Thirds end at 2^-133 = 1e-40: a value at 1e-36 keeps 13 to 16 of its 24 bits in them.
SMALL_BESIDE_LARGE = {
    "scores of tiny rows and huge keys": (lambda x: (_times(x, 1e-36, "q", "r"), _times(x, 1e36, "k")), [("o",), ("dq",), ("dr",), ("dk",), ("dv",)]),
    "scores of huge rows and tiny keys": (lambda x: (_times(x, 1e36, "q", "r"), _times(x, 1e-36, "k")), [("o",), ("dq",), ("dr",), ("dk",), ("dv",)]),
    "a tiny probe alone": (lambda x: (_times(x, 1e-37, "r"), _times(x, 1e15, "k"), _times(x, 1e-15, "q")), [("o",), ("dq",), ("dr",), ("dk",), ("dv",)]),
    "tiny upstream, huge values": (lambda x: (_times(x, 1e-36, "g"), _times(x, 1e36, "v")), [("o",), ("dq",), ("dr",), ("dk",)]),
    "huge upstream, tiny values": (lambda x: (_times(x, 1e36, "g"), _times(x, 1e-36, "v")), [("dq",), ("dr",), ("dk",), ("dv",)]),
    "one tiny column of v": (lambda x: x["v"][..., 5].mul_(1e-36), [("o",), ("o", Ellipsis, 5), ("dq",), ("dv",)]),
    "one tiny row of dO": (lambda x: x["g"][:, :, 70].mul_(1e-36), [("dq",), ("dq", 70), ("dr", 70), ("dk",), ("dv",)]),
    "a tiny row of q, a huge dimension of k": (lambda x: (x["q"][..., 3].mul_(1e-36), x["q"][:, :, 70, :3].zero_(), x["q"][:, :, 70, 4:].zero_(),
                                                         x["r"][..., 3].mul_(1e-36), x["k"][..., 3].mul_(1e36)), [("o",), ("o", 70), ("dr", 70)]),
    "weights of tiny factors, huge rows": (lambda x: (_times(x, 1e-25, "g"), _times(x, 1e-10, "v"), _times(x, 1e20, "q", "r"),
                                                      _times(x, 1e-20, "k")), [("o",), ("dk",), ("dv",)]),
    "weights of tiny factors, huge keys": (lambda x: (_times(x, 1e-25, "g"), _times(x, 1e-10, "v"), _times(x, 1e-20, "q", "r"),
                                                      _times(x, 1e20, "k")), [("o",), ("dq",), ("dr",), ("dv",)]),
    "zeros among them": (lambda x: (_times(x, 1e-36, "q", "r"), _times(x, 1e36, "k"), x["k"][:, :, ::3].zero_(), x["q"][..., ::5].zero_(),
                                    x["v"][:, :, :, 7].zero_(), x["g"][:, :, ::7].zero_()), [("o",), ("dq",), ("dr",), ("dk",), ("dv",)]),
}


@pytest.mark.parametrize("what", list(SMALL_BESIDE_LARGE))
def test_small_values_beside_large_ones(plx, what):
    """Values that three thirds do not hold, times large ones or next to ordinary ones: no less exact than elsewhere."""
    from oracle import parallax_backward

    scale, looked_at = SMALL_BESIDE_LARGE[what]
    x = _inputs(4, 32, 32, 230, 230, seed=31)
    assert _forms(plx, x) == (32, 32, 32)
    scale(x)
    outs = _step(plx, x)
    one = _one_head(x, 2, 7)
    few = _step(plx, one)
    args = [host(one[n]) for n in "qrkv"]
    want = [parallax_backward.forward_with_cache(*args, 0.125)[0], *parallax_backward.backward(*args, host(one["g"]), 0.125)]
    names = ("o", "dq", "dr", "dk", "dv")
    bad = []
    for name, *part in looked_at:
        at = (0, 0, *part)
        got, fp32, ref = (np.asarray(t[names.index(name)], np.float64)[at] for t in
                          ([host(t) for t in _head_of(outs, 2, 7, 1)], [host(t) for t in few], want))
        size = np.abs(ref).max()
        errs = [rel_l2(t / size, ref / size) for t in (got, fp32)]
        print(what, name, part, "%.2g, fp32 instruction %.2g" % tuple(errs))
        if errs[0] > max(REL, 1.5 * errs[1]):
            bad.append((name, part, errs))
    assert not bad


@pytest.mark.parametrize("bad", [math.nan, math.inf, -math.inf])
@pytest.mark.parametrize("name", list("qrkvg"))
@pytest.mark.parametrize("window,G", [(0, 1), (100, 1), (0, 2)])
def test_not_finite_as_the_fp32_kernels_have_it(plx, name, bad, window, G):
    """One value that is not finite: the results are infinite or NaN where those of the fp32 kernels are, and as
    close to them as ever everywhere else."""
    x = _inputs(4, 32 * G, 32, 230, 230, seed=21)
    assert _forms(plx, x, window=window) == (32, 32, 32)
    x[name][2, 7 if name in "kv" else 7 * G + G - 1, 70, 3] = bad
    outs, few = _step(plx, x, window=window), _step(plx, _one_head(x, 2, 7), window=window)
    for n, got, ref in zip(("o", "dq", "dr", "dk", "dv"), _head_of(outs, 2, 7, G), few):
        a, b = host(got).astype(np.float64), host(ref).astype(np.float64)
        ok = np.isfinite(b)
        assert (np.isfinite(a) == ok).all(), n
        if n != "dk":  # (there two infinities may meet in either order)
            assert np.array_equal(a[~ok], b[~ok], equal_nan=True), n
        if ok.any():
            assert rel_l2(a[ok], b[ok]) <= 2 * REL, n
    rest = _step(plx, _one_head(x, 1, 7), window=window)
    for got, ref in zip(_head_of(outs, 1, 7, G), rest):
        assert rel_l2(host(got), host(ref).astype(np.float64)) <= 2 * REL


@pytest.mark.parametrize("what", ["peaked", "one sign"])
def test_peaked_scores_and_values_of_one_sign(plx, what):
    """Scores of up to 40 (their rounding, 2^-24 of them, is what the weights are off by), and values in [0, 1), whose products
    add up: u = rho.k and a = dO.v are 16 on average, so that o = (1 + ubar) vbar - sum p u v is what is left of 16 times its
    size, and tau = dO.o, 16 too, is off by 16 times the error of o; a gradient, sums of p (a - tau) k whose p add up to 1,
    by half of that (k is 1/2 on average) on top."""
    from oracle import parallax_backward

    x = _inputs(4, 32, 32, 257, 257, seed=41)
    if what == "peaked":
        x["q"] *= 6
    else:
        gen = torch.Generator(device=DEV).manual_seed(42)
        x = {n: torch.rand(t.shape, generator=gen, device=DEV) for n, t in x.items()}
    assert _forms(plx, x) == (32, 32, 32)
    outs, one = _step(plx, x), _one_head(x, 1, 9)
    few, args = _step(plx, one), [host(one[n]) for n in "qrkv"]
    want = [parallax_backward.forward_with_cache(*args, 0.125)[0], *parallax_backward.backward(*args, host(one["g"]), 0.125)]
    top = float((one["q"] @ one["k"].transpose(2, 3)).abs().max()) * 0.125
    off = rel_l2(host(few[0]), want[0])
    for name, got, fp32, ref in zip(("o", "dq", "dr", "dk", "dv"), _head_of(outs, 1, 9, 1), few, want):
        errs = rel_l2(host(got), ref), rel_l2(host(fp32), ref)
        bound = max(REL, 4 * top * 2 ** -24) if what == "peaked" else 16 * REL + 8 * off / float(np.sqrt(np.mean(ref ** 2)))
        print(what, name, "%.2g, fp32 instruction %.2g" % errs, "bound %.2g" % bound)
        assert errs[0] <= bound and errs[0] <= 1.5 * errs[1], (name, errs, bound)
