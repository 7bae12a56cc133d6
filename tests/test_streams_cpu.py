"""What a call allocates, and from whose memory where it goes to another stream. The entry points are run with the launches and the streams
replaced by records, on host tensors that pass for device tensors: whatever a call allocates for
a launch stream has to come from that stream's memory (or be told to the allocator, with the launch
waiting for the stream that it came from)."""
import contextlib
import types

import pytest
import torch


class Dev(torch.Tensor):
    """A host tensor that says it is on the device."""

    is_cuda = property(lambda self: True)

    def record_stream(self, stream):
        self.told = getattr(self, "told", ()) + (stream.cuda_stream,)


def dev(*shape, dtype=torch.bfloat16):
    return torch.zeros(*shape, dtype=dtype).as_subclass(Dev)


class Stream(types.SimpleNamespace):
    def wait_stream(self, other):
        self.waited.append(other.cuda_stream)


@pytest.fixture()
def world(monkeypatch):
    """binding with stream 1 as the current one, launches on stream 2, and the list of allocations."""
    from paper_2605_29157_amd import binding

    lib = binding.load_library()
    streams = {i: Stream(cuda_stream=i, waited=[]) for i in (1, 2)}
    now, made, launches = [1], [], []

    @contextlib.contextmanager
    def use(stream):
        now.append(stream.cuda_stream)
        yield
        now.pop()

    def recorded(make):
        def wrapped(*args, **kw):
            kw.pop("device", None)
            t = make(*args, **kw).as_subclass(Dev)
            made.append((now[-1], t))
            return t
        return wrapped

    class Lib:
        def __getattr__(self, name):
            if name.endswith(("bytes", "splits")):
                return getattr(lib, name)
            return lambda *args: launches.append((name, args[-1])) or 0

    monkeypatch.setattr(binding, "load_library", lambda: Lib())
    monkeypatch.setattr(binding, "_stream_ptr", lambda s: now[-1] if s is None else s.cuda_stream)
    monkeypatch.setattr(torch.cuda, "stream", use)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: streams[now[-1]])
    monkeypatch.setattr(torch.cuda, "ExternalStream", lambda ptr, device=None: streams[ptr])
    monkeypatch.setattr(torch, "empty", recorded(torch.empty))
    monkeypatch.setattr(torch, "empty_like", recorded(torch.empty_like))
    monkeypatch.setattr(torch, "empty_strided", recorded(torch.empty_strided))
    return types.SimpleNamespace(plx=binding, streams=streams, made=made, launches=launches)


def _prefill(w, T, Tkv, **kw):
    q, r, k, v = dev(1, 2, T, 128), dev(1, 2, T, 128), dev(1, 2, Tkv, 128), dev(1, 2, Tkv, 128)
    return w.plx.parallax_prefill(q, r, k, v, 0.1, stream=w.streams[2], **kw)


def _decode(w, dtype, **kw):
    q, r, k, v = dev(1, 4, 64, dtype=dtype), dev(1, 4, 64, dtype=dtype), *(dev(1, 2, 4096, 64, dtype=dtype) for _ in "kv")
    return w.plx.parallax_decode(q, r, k, v, 0.1, stream=w.streams[2], **kw)


def _backward(w, **kw):
    x = [dev(1, 2, 256, 128) for _ in range(7)]
    return w.plx.parallax_prefill_backward(*x[:6], dev(1, 2, 256, 2, dtype=torch.float32), x[6], 0.1, stream=w.streams[2], **kw)


MASK = torch.ones(2, 4, dtype=torch.bool).as_subclass(Dev)
CALLS = {
    "decode_bf16": lambda w: _decode(w, torch.bfloat16),
    "decode_f32": lambda w: _decode(w, torch.float32),
    "decode_own_output": lambda w: _decode(w, torch.float32, out=dev(1, 4, 64, dtype=torch.float32)),
    "mla": lambda w: w.plx.parallax_decode_mla(dev(1, 16, 576), dev(1, 16, 576), dev(1, 4096, 576), 0.1, stream=w.streams[2]),
    "prefill_split": lambda w: _prefill(w, 64, 8192),
    "prefill_cache": lambda w: _prefill(w, 64, 64, save_for_backward=True),
    "prefill_mask": lambda w: _prefill(w, 256, 256, block_mask=MASK),
    "backward": lambda w: _backward(w),
    "backward_mask": lambda w: _backward(w, block_mask=MASK),
    "norm_rope": lambda w: w.plx.parallax_norm_rope([(dev(1, 2, 3, 64), dev(64, dtype=torch.float32), True)], stream=w.streams[2]),
    "rope_table": lambda w: w.plx.parallax_rope_table(4, 64, stream=w.streams[2]),
}


@pytest.mark.parametrize("name", CALLS)
def test_memory_of_a_call_on_another_stream(world, name):
    result = CALLS[name](world)
    assert world.made and world.launches[-1][1] == 2
    returned = [t for t in (result if isinstance(result, (tuple, list)) else [result])]
    for stream, t in world.made:
        told = getattr(t, "told", ())
        if stream == 2:  # its own memory; what the caller gets is used on the caller's stream too
            assert any(t is x for x in returned) == (1 in told)
        else:  # the lists of a block mask: built on the current stream, where the mask is
            assert "mask" in name and t.dtype == torch.int32
            assert told == (2,) and world.streams[2].waited == [1]
            assert world.launches[0] == ("parallax_block_lists", 1)
    assert any(t.dtype == torch.float32 and not any(t is x for x in returned) for _, t in world.made) == (
        name in ("decode_bf16", "decode_f32", "decode_own_output", "mla", "prefill_split", "backward", "backward_mask"))


@pytest.mark.parametrize("B,Hq,Hkv,Tq,L,window,records", [
    (64, 32, 8, 1, 16384, 0, 0),         # workgroups for every compute unit twice: unsplit
    (1, 16, 8, 4096, 16384, 0, 0),       # so have many query rows
    (1, 16, 8, 1, 16384, 256, 16 * 2),   # two splits of 128 keys inside the window
    (1, 16, 8, 1, 16384, 0, 16 * 64),    # 512 workgroups for 256 compute units
    (2, 4, 4, 1, 200, 0, 0)])
def test_fp32_decode_allocates_the_records_that_it_uses(world, B, Hq, Hkv, Tq, L, window, records):
    q = dev(B, Hq, Tq, 64, dtype=torch.float32) if Tq > 1 else dev(B, Hq, 64, dtype=torch.float32)
    k = dev(1, 1, L, 64, dtype=torch.float32).expand(B, Hkv, L, 64)
    world.plx.parallax_decode(q, q, k, k, 0.1, window=window, out=q)
    assert sum(t.numel() for _, t in world.made) == records * (2 * 64 + 4)


def test_split_count_of_a_call(world):
    """bf16: the pick of the shape query; explicit counts; 0 for arguments that the call would refuse."""
    import ctypes

    lib = world.plx.load_library()
    q, k = dev(1, 16, 128), dev(1, 8, 16384, 128)
    for kw, want in ((dict(), lib.parallax_decode_num_splits(1, 16, 8, 16384, 128, 0)), (dict(num_splits=3), 3),
                     (dict(window=2000), lib.parallax_decode_num_splits(1, 16, 8, 2000, 128, 0)), (dict(num_splits=129), 0)):
        a = world.plx.decode_args(q, q, k, k, q, 0.1, **kw)
        a.o = None
        assert lib.parallax_decode_call_splits(ctypes.byref(a)) == want


@pytest.mark.parametrize("columns", [False, True])
def test_masks_that_the_list_kernels_do_not_take(world, monkeypatch, columns):
    """Beyond the lines that parallax_block_lists accepts, the lists come from tensor operations."""
    monkeypatch.setattr(world.plx, "_MAX_LIST_LINES", 27)  # (7 lines per list)
    mask = (torch.arange(2 * 4 * 5) % 3 == 0).reshape(2, 1, 4, 5)
    a = (world.plx.plx_prefill_bwd_args if columns else world.plx.plx_prefill_args)()
    world.plx.attach_block_lists(a, mask[:1], "cpu", columns=columns)
    assert [name for name, _ in world.launches] == ["parallax_block_lists"]
    held = world.plx.attach_block_lists(a, mask.repeat(2, 1, 1, 1), "cpu", world.streams[1], columns)
    assert len(world.launches) == 1 and (a.sparse_batch, a.sparse_heads) == (4, 1)
    want = world.plx.block_mask_lists(mask.repeat(2, 1, 1, 1))[:2]
    want += world.plx.block_mask_column_lists(mask.repeat(2, 1, 1, 1)) if columns else ()
    assert len(held) == len(want) and all(torch.equal(x, y) for x, y in zip(held, want))
    assert [t.data_ptr() for t in held[:2]] == [a.sparse_row_ptr, a.sparse_tile_idx]
    if columns:
        assert [t.data_ptr() for t in held[2:]] == [a.sparse_col_ptr, a.sparse_col_idx]


def test_the_row_cache_is_laid_out_like_an_output_with_gaps(world):
    """The kernel writes vbar with the strides of out: so it has to have them, where out is every second row
    of a larger tensor (bytes behind a dense vbar's end would be written otherwise)."""
    q, out = dev(1, 2, 8, 64), dev(1, 2, 16, 64)[:, :, ::2]
    for stream in (None, world.streams[2]):
        got, vbar, _ = world.plx.parallax_prefill(q, q, q, q, 0.1, out=out, save_for_backward=True, stream=stream)
        assert got is out and vbar.stride() == out.stride() and vbar.shape == out.shape
