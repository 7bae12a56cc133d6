"""Calls on another stream than the current one, without a workspace, between work of the current stream on
memory of the same sizes: freed in front of the call with writes to it still queued, and
allocated and written right behind it. The results are those of the call on the current stream."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def plx():
    from paper_2605_29157_amd import binding

    binding.load_library()
    return binding


def _rand(*shape, dtype=torch.bfloat16):
    gen = torch.Generator(device=DEV).manual_seed(sum(shape))
    return torch.randn(shape, generator=gen, device=DEV).to(dtype)


def _calls(plx):
    def decode(dtype, **kw):
        q, r = _rand(2, 8, 128, dtype=dtype), _rand(2, 8, 128, dtype=dtype)
        k, v = _rand(2, 4, 6000, 128, dtype=dtype), _rand(2, 4, 6001, 128, dtype=dtype)[:, :, :6000]
        return lambda stream: plx.parallax_decode(q, r, k, v, 0.09, stream=stream, **kw)

    def mla():
        q, r, c = _rand(2, 16, 576), _rand(2, 16, 576), _rand(2, 4000, 576)
        return lambda stream: plx.parallax_decode_mla(q, r, c, 0.04, stream=stream)

    def prefill(T, Tkv, **kw):
        q, r, k, v = _rand(1, 4, T, 128), _rand(1, 4, T, 128), _rand(1, 2, Tkv, 128), _rand(1, 2, Tkv, 128)
        return lambda stream: plx.parallax_prefill(q, r, k, v, 0.09, stream=stream, **kw)

    def backward(**kw):
        q, r, g = (_rand(1, 4, 700, 128) for _ in range(3))
        k, v = _rand(1, 2, 700, 128), _rand(1, 2, 700, 128)
        o, vbar, st = plx.parallax_prefill(q, r, k, v, 0.09, save_for_backward=True, **kw)
        return lambda stream: plx.parallax_prefill_backward(q, r, k, v, o, vbar, st, g, 0.09, stream=stream, **kw)

    mask = torch.ones(6, 11, dtype=torch.bool, device=DEV)
    return {"decode_bf16": decode(torch.bfloat16), "decode_f32": decode(torch.float32), "mla": mla(),
            "prefill_split": prefill(64, 8000), "prefill_cache": prefill(200, 3000, save_for_backward=True),
            "prefill_mask": prefill(700, 700, block_mask=mask), "backward": backward(),
            "backward_mask": backward(block_mask=mask)}


def _noise():
    """Blocks of every size class of the allocator, written on the current stream."""
    return [torch.full((n,), float("nan"), device=DEV) for n in (512, 40_000, 300_000, 3_000_000, 20_000_000)]


def test_other_stream_between_busy_memory(plx):
    side = torch.cuda.Stream()
    for name, call in _calls(plx).items():
        want = call(None)
        torch.cuda.synchronize()
        blocks = _noise()
        torch.cuda._sleep(3_000_000)
        for b in blocks:
            b.fill_(float("nan"))
        del blocks, b  # free, with the writes still behind the pause
        got = call(side)
        after = _noise()
        torch.cuda.synchronize()
        for a, b in zip(want if isinstance(want, tuple) else (want,), got if isinstance(got, tuple) else (got,)):
            assert torch.equal(a, b), name
        del after


def test_a_result_dropped_while_it_is_read(plx):
    """What the caller gets may be dropped as soon as its own stream has been given the work that reads it."""
    call = _calls(plx)["decode_bf16"]
    want = call(None)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    sums = []
    for _ in range(8):
        got = call(side)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda._sleep(300_000)
        sums.append(got.clone())
        del got
    torch.cuda.synchronize()
    assert all(torch.equal(s, want) for s in sums)
