"""The native marshalling (csrc/binding.cpp) against the ctypes route: the same bits for every form of call both take,
the same exception for what either refuses."""
import pytest
import torch

import paper_2506_11418_amd as ckv

pytestmark = pytest.mark.gpu
DEV = "cuda"


class _Never:
    """Stands for the native module: takes nothing, so every call goes by ctypes."""

    def __getattr__(self, name):
        return lambda *args: None


class _Counting:
    """The native module, counting what it took."""

    def __init__(self, module):
        self.module, self.took = module, 0

    def __getattr__(self, name):
        fn = getattr(self.module, name)

        def call(*args):
            status = fn(*args)
            self.took += status == 0
            return status
        return call


def _both(monkeypatch, make, call, native=True):
    """call(make()) by either route; returns the outputs of the two, checks who made the call."""
    real = ckv._binding()
    outs = []
    for module in (_Counting(real), _Never()):
        monkeypatch.setattr(ckv, "_native", module)
        outs.append([x.clone() if isinstance(x, torch.Tensor) else x for x in call(make())])
        torch.cuda.synchronize()
        if isinstance(module, _Counting):
            assert (module.took > 0) == native
    for a, b in zip(*outs):
        assert torch.equal(a, b) if isinstance(a, torch.Tensor) else a == b
    return outs[0]


def _kv(seed, shape, dtype, order="bhsd"):
    g = torch.Generator(device=DEV).manual_seed(seed)
    b, h, s, d = shape
    if order == "bhsd":
        return [torch.randn(shape, generator=g, device=DEV).to(dtype) for _ in range(2)]
    if order == "bshd":
        return [torch.randn((b, s, h, d), generator=g, device=DEV).to(dtype).transpose(1, 2) for _ in range(2)]
    return [torch.randn((b, h, s + 24, d), generator=g, device=DEV).to(dtype)[:, :, :s] for _ in range(2)]   # spare rows


@pytest.mark.parametrize("order", ["bhsd", "bshd", "spare"])
@pytest.mark.parametrize("dtype,rounds,scope,route,with_deg", [
    (torch.bfloat16, None, "chunk", None, False), (torch.bfloat16, [0.5, 1], "head", None, True),
    (torch.float32, (1.0, 0.25), "chunk", "full_rounds", True), (torch.bfloat16, [1.0, 0.8], "chunk", "defer_always", False),
])
def test_compress_by_either_route(monkeypatch, order, dtype, rounds, scope, route, with_deg):
    print("binding: compress", order, dtype, rounds, scope, route, flush=True)
    B, H, S, D = 2, 3, 700, 64

    def make():
        K, V = _kv(1, (B, H, S, D), dtype, order)
        deg = None
        if with_deg:
            deg = torch.randint(1, 9, (B, H, S + 24), device=DEV, dtype=torch.int32, generator=torch.Generator(device=DEV).manual_seed(2))
            deg = deg[:, :, :S] if order == "spare" else deg[:, :, :S].contiguous()
        kw = dict(chunk=128, rounds=rounds, n_sink=4, n_recent=8, scope=scope, route=route, retain_ratio=0.5 if rounds is None else 1)
        pl = ckv.plan(ckv.layout_of(K, deg), ckv.make_params(**kw))
        out = (torch.zeros((B, H, pl.out_seq + 5, D), dtype=dtype, device=DEV), torch.zeros((B, H, pl.out_seq + 5, D), dtype=dtype, device=DEV),
               torch.zeros((B, H, pl.out_seq + 5), dtype=torch.int32, device=DEV), torch.zeros((B, H, S), dtype=torch.int32, device=DEV))
        return K, V, dict(kw, deg=deg, out=out, workspace=torch.zeros(max(pl.workspace_bytes, 256), dtype=torch.uint8, device=DEV))
    _both(monkeypatch, make, lambda x: ckv.compress(x[0], x[1], **x[2]))


@pytest.mark.parametrize("order", ["bhsd", "bshd", "spare"])
@pytest.mark.parametrize("dtype,batch,with_deg,with_lens", [(torch.bfloat16, 1, True, False), (torch.float32, 3, False, True),
                                                            (torch.bfloat16, 2, True, True)])
def test_append_and_attention_by_either_route(monkeypatch, order, dtype, batch, with_deg, with_lens):
    print("binding: append, attention", order, dtype, batch, flush=True)
    H, S, D, G = 2, 90, 64, 4

    def make():
        K, V = _kv(3, (batch, H, S, D), dtype, order)
        deg = torch.ones((batch, H, S), dtype=torch.int32, device=DEV) * 3 if with_deg else None
        lens = torch.tensor([40 + 7 * b for b in range(batch)], dtype=torch.int32, device=DEV) if with_lens else None
        q, kn = (_kv(s, (1, batch, n, D), dtype)[0][0] for s, n in ((4, H * G), (5, H)))
        ws = torch.zeros(ckv.decode_attn_workspace(ckv.layout_of(K), H * G), dtype=torch.uint8, device=DEV)
        return K, V, deg, lens, q, kn, kn * 2, torch.zeros((batch, H * G, D), dtype=torch.float32, device=DEV), ws

    def call(x):
        K, V, deg, lens, q, kn, vn, o, ws = x
        ckv.append(kn, vn, K, V, deg, lens=lens, pos=-1 if with_lens else 50)
        ckv.decode_attn(q, K, V, lens=lens, deg=deg, scale=0, out=o, workspace=ws)
        return [o, K, V] + [t for t in (deg, lens) if t is not None]
    _both(monkeypatch, make, call)


def test_paged_calls_by_either_route(monkeypatch):
    print("binding: paged", flush=True)
    B, H, D, bs, G = 2, 2, 128, 16, 2

    def make():
        K, V = _kv(7, (12, H, bs, D), torch.bfloat16)
        table = torch.randperm(12, generator=torch.Generator().manual_seed(1)).to(torch.int32).view(B, 6).to(DEV)
        q, kn = (_kv(s, (1, B, n, D), torch.bfloat16)[0][0] for s, n in ((8, H * G), (9, H)))
        pl = ckv.paged_layout_of(K, table)
        n = ckv.C.c_size_t(0)
        assert ckv.lib().ckv_paged_decode_attn_workspace(ckv.C.byref(pl), H * G, 96, ckv.C.byref(n)) == 0
        return (K, V, torch.ones((12, H, bs), dtype=torch.int32, device=DEV), table, torch.tensor([50, 79], dtype=torch.int32, device=DEV),
                q, kn, torch.zeros_like(q), torch.zeros(n.value, dtype=torch.uint8, device=DEV))

    def call(x):
        K, V, deg, table, lens, q, kn, o, ws = x
        ckv.paged_append(kn, kn, K, V, deg, table, lens)
        ckv.paged_decode_attn(q, K, V, deg, table, lens, 96, out=o, workspace=ws)
        return [o, K, V, deg, lens]
    _both(monkeypatch, make, call)


def test_refused_calls_raise_the_same_by_either_route(monkeypatch):
    print("binding: refusals", flush=True)
    K, V = _kv(1, (1, 2, 64, 64), torch.bfloat16)
    q, kn = torch.zeros((1, 8, 64), dtype=torch.bfloat16, device=DEV), torch.zeros((1, 2, 64), dtype=torch.bfloat16, device=DEV)
    o, ws = torch.zeros_like(q), torch.zeros(ckv.decode_attn_workspace(ckv.layout_of(K), 8), dtype=torch.uint8, device=DEV)
    out = (torch.zeros_like(K), torch.zeros_like(V), torch.zeros((1, 2, 64), dtype=torch.int32, device=DEV), None)
    big = torch.zeros(1 << 20, dtype=torch.uint8, device=DEV)
    calls = [
        lambda: ckv.append(kn[:, :1], kn, K, V, None, pos=3),                              # a head missing
        lambda: ckv.append(kn, kn, K, V, None, pos=64),                                    # behind the capacity
        lambda: ckv.append(kn, kn, K.transpose(2, 3), V.transpose(2, 3), None, pos=0),     # channels apart
        lambda: ckv.decode_attn(q.float(), K, V, out=o, workspace=ws),
        lambda: ckv.decode_attn(q, K, V, out=o, workspace=ws[:64]),                        # workspace too small
        lambda: ckv.decode_attn(q[:, :3], K, V, out=o, workspace=ws),                      # not contiguous heads of a group
        lambda: ckv.decode_attn(q, K, V, out=o.half(), workspace=ws),
        lambda: ckv.decode_attn(q, K, V, deg=torch.ones((1, 2, 63), dtype=torch.int32, device=DEV), out=o, workspace=ws),
        lambda: ckv.compress(K, V, 63, rounds=[1.0], out=out, workspace=big),              # odd chunk
        lambda: ckv.compress(K, V.float(), 64, rounds=[1.0], out=out, workspace=big),
        lambda: ckv.compress(K, V, 64, rounds=[], out=out, workspace=big),
        lambda: ckv.compress(K, V, 64, rounds=[1.5], out=out, workspace=big),
        lambda: ckv.compress(K, V, 64.5, rounds=[1.0], out=out, workspace=big),
        lambda: ckv.compress(K, V, 64, rounds=[1.0], scope="cluster", out=out, workspace=big),
        lambda: ckv.compress(K, V, 64, rounds=[1.0], out=(K,) + out[1:], workspace=big),   # in place
        lambda: ckv.compress(K, V, 64, rounds=[1.0], out=out, workspace=big[1:]),          # misaligned
    ]
    for i, call in enumerate(calls):
        kinds = []
        for module in (ckv._binding(), _Never()):
            monkeypatch.setattr(ckv, "_native", module)
            with pytest.raises(Exception) as e:
                call()
            kinds.append((e.type, str(e.value)))
            monkeypatch.undo()
        assert kinds[0] == kinds[1], (i, kinds)
