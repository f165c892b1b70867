"""What the Python entry points do with the native binding's answer, without a GPU: None goes on to the ctypes route, a
status ends the call."""
import pytest
import torch

import paper_2506_11418_amd as ckv

B, H, S, D, BLOCK = 1, 2, 64, 64, 16


class _OnGpu(torch.Tensor):
    """A host tensor that says it lives on the GPU; nothing here follows its pointer."""
    is_cuda = property(lambda self: True)


def _t(*shape, dtype=torch.bfloat16):
    return torch.zeros(shape, dtype=dtype).as_subclass(_OnGpu)


class _Answer:
    """Stands for the native module: every call answers `status`."""

    def __init__(self, status):
        self.status = status

    def __getattr__(self, name):
        return lambda *args: self.status


class _Calls:
    """Stands for the library: answers CKV_OK and counts; what computes sizes or texts is the real one."""

    def __init__(self, real):
        self.real, self.made = real, 0

    def __getattr__(self, name):
        if name in ("ckv_strerror", "ckv_plan"):
            return getattr(self.real, name)

        def call(*args):
            self.made += 1
            return 0
        return call


def _calls():
    K, V, deg, lens = _t(B, H, S, D), _t(B, H, S, D), _t(B, H, S, dtype=torch.int32), _t(B, dtype=torch.int32)
    kn, q, o, ws = _t(B, H, D), _t(B, H, D), _t(B, H, D), _t(1 << 20, dtype=torch.uint8)
    pool, dpool, table = _t(4, H, BLOCK, D), _t(4, H, BLOCK, dtype=torch.int32), _t(B, 4, dtype=torch.int32)
    out = (_t(B, H, S, D), _t(B, H, S, D), _t(B, H, S, dtype=torch.int32), None)
    return {
        "ckv_append": lambda: ckv.append(kn, kn, K, V, deg, lens=lens),
        "ckv_paged_append": lambda: ckv.paged_append(kn, kn, pool, pool, dpool, table, lens),
        "ckv_decode_attn": lambda: ckv.decode_attn(q, K, V, lens=lens, out=o, workspace=ws),
        "ckv_paged_decode_attn": lambda: ckv.paged_decode_attn(q, pool, pool, dpool, table, lens, S, out=o, workspace=ws),
        "ckv_compress": lambda: ckv.compress(K, V, 64, rounds=[1.0], out=out, workspace=ws),
    }


@pytest.fixture
def library(monkeypatch):
    stub = _Calls(ckv.lib())
    monkeypatch.setattr(ckv, "lib", lambda: stub)
    monkeypatch.setattr(ckv, "_raw_stream", lambda: 0)
    monkeypatch.setattr(ckv, "_stream", lambda: None)
    return stub


@pytest.mark.parametrize("name", list(_calls()))
@pytest.mark.parametrize("status", [-6, -5, -2])     # (a status of the runtime: the launch may have been made)
def test_a_call_that_was_made_is_not_made_again(monkeypatch, library, name, status):
    monkeypatch.setattr(ckv, "_native", _Answer(status))
    with pytest.raises(ckv.CkvError) as e:
        _calls()[name]()
    assert e.value.status == status and str(e.value).startswith(name + ":")
    assert library.made == 0


@pytest.mark.parametrize("name", list(_calls()))
def test_a_call_the_binding_does_not_take_is_made_once(monkeypatch, library, name):
    monkeypatch.setattr(ckv, "_native", _Answer(None))
    _calls()[name]()
    assert library.made == 1


@pytest.mark.parametrize("rounds,error", [((x for x in (1.0,)), TypeError), ({1.0: 1}, None), ({1.0}, None), ((1.0,), None), ([1.0], None)])
def test_rounds_the_binding_does_not_know_go_to_ctypes_unread(monkeypatch, library, rounds, error):
    """Whatever has a length and an order of its own is taken as before, and a generator is refused as before."""
    class _Lists:
        def compress(self, *args):
            return 0 if args[5] is None or type(args[5]) is list else None
    monkeypatch.setattr(ckv, "_native", _Lists())
    K, ws = _t(B, H, S, D), _t(1 << 20, dtype=torch.uint8)
    out = (_t(B, H, S, D), _t(B, H, S, D), _t(B, H, S, dtype=torch.int32), None)
    call = lambda: ckv.compress(K, K, 64, rounds=rounds, out=out, workspace=ws)
    if error:
        with pytest.raises(error):
            call()
    else:
        call()
    assert library.made == (not error and not isinstance(rounds, (list, tuple)))
