"""The native argument checks of the Python binding: they make the call for good arguments and leave
everything else (None) to the Python checks, which raise."""

import ctypes

import pytest
import torch

from paper_2510_13223_amd import bana, workloads as W


def test_native_checks_leave_host_arguments_to_python():
    n = bana._calls()
    cpu = torch.zeros(2, 2, 128)
    assert n.partial(*[cpu] * 9, None, None, None, 0) is None
    assert n.noalloc(*[cpu] * 9, None, None, 0) is None
    assert n.fused(*[cpu] * 9, None, None, None, None) is None
    assert n.heads(*[cpu] * 7, 0, 1, cpu, cpu, None, None, None) is None
    assert n.merge(cpu, cpu, cpu, None, None) is None
    assert n.migrate(*[cpu] * 8, None, 0) is None
    assert n.partial(1, 2, 3) is None and n.merge() is None
    with pytest.raises(TypeError):
        n.setup(1, 2, 3, 4)
    with pytest.raises((TypeError, ValueError)):
        bana.bana_merge_partials(torch.zeros(2, 1, 1, 128), torch.zeros(2, 1, 1), cpu)


@pytest.fixture
def without_native(monkeypatch):
    """Only the C library built, as by `make`: the import of the native module fails."""
    import sys

    import paper_2510_13223_amd as pkg

    monkeypatch.setattr(bana, "_native", None)
    monkeypatch.delattr(pkg, "_native", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2510_13223_amd._native", None)


def test_binding_works_without_the_native_checks(without_native):
    with pytest.warns(RuntimeWarning, match="make binding"):
        n = bana._calls()
    assert n.merge(1, 2, 3, None, None) is None and bana._calls() is n
    with pytest.raises(ValueError):
        bana.bana_merge_partials(torch.zeros(2, 1, 1, 128), torch.zeros(2, 1, 1), torch.zeros(1, 1, 128))


@pytest.mark.gpu
@pytest.mark.filterwarnings("ignore:the native argument checks")
def test_calls_without_the_native_checks_have_the_same_results(without_native):
    from paper_2510_13223_amd.runner import DeviceWorkload

    w = W.make_config("tiny", 0)
    plain = DeviceWorkload(w).results()
    bana._native = None
    import sys

    del sys.modules["paper_2510_13223_amd._native"]
    for a, b in zip(plain, DeviceWorkload(w).results()):
        assert (a == b).all()
    assert not isinstance(bana._calls(), bana._PythonChecks)


@pytest.mark.gpu
def test_native_checks_take_good_arguments_and_refuse_bad_ones():
    from paper_2510_13223_amd.runner import DeviceWorkload

    w = W.make_config("tiny", 0)
    dw = DeviceWorkload(w)
    n = bana._calls()
    side = torch.cuda.Stream()
    ws = torch.empty(1 << 22, dtype=torch.uint8, device="cuda")
    args = [dw.q, dw.k_cache, dw.v_cache, dw.block_table, dw.seq_lens, dw.kv_begin[0], dw.kv_end[0],
            dw.out_partials[0], dw.lses[0]]
    fused = args[:5] + [dw.kv_begin, dw.kv_end, dw.fused_out, dw.fused_lse]
    torch.cuda.synchronize()
    for stream in (None, 0, side, side.cuda_stream):
        for dims in (None, dw.dims[0]):
            assert n.partial(*args, ws, stream, dims, 0) == 0
            assert n.noalloc(*args, stream, dims, 0) == 0
            assert n.fused(*fused, None, stream, dims, None) == 0
            assert n.fused(*fused, None, stream, dims, []) == 0
            assert n.heads(*args[:7], 0, 1, *args[7:], ws, stream, dims) == 0
            torch.cuda.synchronize()
    assert n.merge(dw.out_partials, dw.lses, dw.out, dw.lse_out, None) == 0
    assert n.merge(dw.out_partials, dw.lses, dw.out, None, None) == 0
    dst = [torch.zeros_like(dw.k_cache), torch.zeros_like(dw.v_cache)]
    zero = torch.zeros_like(dw.seq_lens)
    assert n.migrate(dw.k_cache, dw.v_cache, dw.block_table, *dst, dw.block_table, zero, zero, None, 0) == 0

    class Sub(torch.Tensor):
        pass

    # One bad argument at a time: another type, dtype, shape, layout, device, a subclass.
    for i in range(len(args)):
        t = args[i]
        bad = [None, 3, t.double(), t.cpu(), t[:0] if t.dim() == 1 else t[..., :1], t.as_subclass(Sub)]
        if t.dim() > 1:
            bad.append(t.transpose(0, 1))
        for x in bad:
            assert n.partial(*args[:i], x, *args[i + 1:], ws, None, None, 0) is None, (i, type(x))
    wrong = bana.bana_dims.from_buffer_copy(dw.dims[0])
    wrong.num_blocks += 1
    for dims in (wrong, object(), (ctypes.c_char * ctypes.sizeof(wrong))()):
        assert n.partial(*args, ws, None, dims, 0) is None
        with pytest.raises((ValueError, AttributeError)):
            bana.bana_decode_attn_partial(*args, workspace=ws, dims=dims)
    assert n.partial(*args, ws.cpu(), None, None, 0) is None
    assert n.partial(*args, ws, "stream", None, 0) is None
    # What the library refuses comes back as its status.
    refused = bana.bana_dims.from_buffer_copy(dw.dims[0])
    refused.waves_hint = 3
    assert n.partial(*args, ws, None, refused, 0) == bana.BANA_ERR_INVALID
    # Copies: pairs of one size, on the device or pinned.
    a, b = torch.arange(64, device="cuda", dtype=torch.int32), torch.zeros(64, device="cuda", dtype=torch.int32)
    pinned = torch.zeros(64, dtype=torch.int32).pin_memory()
    assert n.fused(*fused, None, None, None, [(b, a), (pinned, a)]) == 0
    torch.cuda.synchronize()
    assert torch.equal(a, b) and torch.equal(pinned, a.cpu())
    for pair in ((b, a[:32]), (torch.zeros(64, dtype=torch.int32), a), (b[::2], a[:32]), (b,), [b, a]):
        assert n.fused(*fused, None, None, None, [pair]) is None
