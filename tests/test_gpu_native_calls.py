"""The native call path of the binding against its general path: the same bits for what it takes, the same errors for
what it leaves to the general path, on the current and on a given stream."""
import numpy as np
import pytest
import torch

import kvc_workloads as W
from gpu_util import dev_tensor, out_bits, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture
def K(monkeypatch):
    import paper_2503_13773_amd as K
    from paper_2503_13773_amd import binding as B
    counted = {"native": 0}
    native = B._calls()

    class Counting:
        def __getattr__(self, name):
            f = getattr(native, name)

            def call(*a):
                rc = f(*a)
                counted["native"] += rc is not None
                return rc
            return call
    monkeypatch.setattr(B, "_native", Counting())
    K_ = type("K_", (), dict(K.__dict__, counted=counted, general=lambda: monkeypatch.setattr(B, "_on_device", lambda t: False)))
    return K_


def calls(K, w, stream):
    """Every call once, on fresh outputs; what they wrote."""
    d = to_device(w)
    bf = w.dtype == W.BF16
    desc = K.attn_desc(d["q"], d["k"], d["tables"], max_context_len=w.max_context_len)
    ws = K.new_workspace(desc)
    torch.cuda.synchronize()
    k, v = d["k"].clone(), d["v"].clone()
    rng = np.random.default_rng(5)
    new = [dev_tensor(W._normal(rng, (w.num_seqs, w.num_kv_heads, w.head_dim), w.dtype), w.dtype) for _ in range(2)]
    pool, second = torch.stack([k, v]), torch.zeros((2, 9) + tuple(k.shape[1:]), dtype=k.dtype, device="cuda")
    m = torch.tensor([[3, 8], [0, 2], [5, 0]], dtype=torch.int64, device="cuda")
    qs = torch.arange(w.num_seqs + 1, dtype=torch.int32, device="cuda")
    outs = [torch.zeros_like(d["q"]) for _ in range(3)]
    torch.cuda.synchronize()
    K.kv_cache_append(new[0], new[1], k, v, d["tables"], d["lens"] - 1, stream=stream)
    K.paged_attention_decode(d["q"], k, v, d["tables"], d["lens"], w.scale, outs[0], desc=desc, workspace=ws, stream=stream)
    K.paged_attention_prefill(d["q"], k, v, d["tables"], d["lens"], qs, w.scale, 1, outs[1], stream=stream)
    K.kv_block_copy(pool, second, m, stream=stream)
    if bf:
        sched = torch.empty(K.schedule_bytes(desc), dtype=torch.uint8, device="cuda")
        K.attn_schedule_build(d["tables"], d["lens"], desc, sched, stream=stream)
        K.paged_attention_decode_scheduled(d["q"], k, v, sched, w.scale, outs[2], desc, ws, stream=stream)
    torch.cuda.synchronize()
    return [out_bits(x) for x in (k, v, second, *outs)]


@pytest.mark.parametrize("name", ["cfg1", "cfg3"])
@pytest.mark.parametrize("side_stream", [False, True])
def test_native_and_general_path_write_the_same(K, name, side_stream):
    w = W.make_config(name, num_seqs=5, ctx_scale=0.5)
    print(f"[case] native calls {name} side stream {side_stream}", flush=True)
    stream = torch.cuda.Stream() if side_stream else None
    got = calls(K, w, stream)
    assert K.counted["native"] == (6 if name == "cfg3" else 4)
    K.general()
    want = calls(K, w, stream)
    assert K.counted["native"] == (6 if name == "cfg3" else 4)
    assert all(np.array_equal(a, b) for a, b in zip(got, want))


def test_what_the_native_path_does_not_take_raises_as_before(K):
    w = W.make_config("cfg3", num_seqs=3, ctx_scale=0.2)
    d = to_device(w)
    out = torch.empty_like(d["q"])
    ok = dict(q=d["q"], k_cache=d["k"], v_cache=d["v"], block_tables=d["tables"], context_lens=d["lens"], scale=w.scale, out=out)
    bad = [dict(q=d["q"].transpose(0, 1)), dict(k_cache=d["k"].cpu()), dict(v_cache=d["v"][:-1].contiguous()),
           dict(v_cache=d["v"].float()), dict(block_tables=d["tables"].long()), dict(context_lens=d["lens"].long()),
           dict(context_lens=d["lens"][:2].contiguous()), dict(out=out.float()), dict(out=out[:, ::2]), dict(q=d["q"].half())]
    seen = []
    for general in (False, True):
        if general:
            K.general()
        for b in bad:
            with pytest.raises((ValueError, TypeError)) as e:
                K.paged_attention_decode(**{**ok, **b}, max_context_len=w.max_context_len)
            seen.append((type(e.value), str(e.value)))
    assert seen[:len(bad)] == seen[len(bad):]
    assert K.counted["native"] == 0


def test_status_codes_become_the_same_error(K):
    w = W.make_config("cfg3", num_seqs=3, ctx_scale=0.2)
    d = to_device(w)
    desc = K.attn_desc(d["q"], d["k"], d["tables"], max_context_len=w.max_context_len)
    out, small = torch.empty_like(d["q"]), torch.zeros(256, dtype=torch.uint8, device="cuda")
    seen = []
    for general in (False, True):
        if general:
            K.general()
        with pytest.raises(K.KvcError) as e:
            K.paged_attention_decode(d["q"], d["k"], d["v"], d["tables"], d["lens"], w.scale, out, desc=desc, workspace=small)
        seen.append((e.value.status, str(e.value)))
    assert seen[0] == seen[1] and seen[0][0] == -5


def test_subclasses_and_functional_transforms_take_the_general_path(K):
    """vmap hands over wrapped tensors without storage of their own: refused as before, never read."""
    w = W.make_config("cfg3", num_seqs=3, ctx_scale=0.2)
    d = to_device(w)
    desc = K.attn_desc(d["q"], d["k"], d["tables"], max_context_len=w.max_context_len)
    ws = K.new_workspace(desc)

    class Sub(torch.Tensor):
        pass
    out = torch.empty_like(d["q"])
    K.paged_attention_decode(d["q"].as_subclass(Sub), d["k"], d["v"], d["tables"], d["lens"], w.scale, out, desc=desc, workspace=ws)
    plain = K.paged_attention_decode(d["q"], d["k"], d["v"], d["tables"], d["lens"], w.scale, torch.empty_like(out), desc=desc,
                                     workspace=ws)
    assert K.counted["native"] == 1 and torch.equal(out, plain)
    with pytest.raises(Exception):
        torch.vmap(lambda q: K.paged_attention_decode(q, d["k"], d["v"], d["tables"], d["lens"], w.scale, out, desc=desc,
                                                      workspace=ws))(torch.stack([d["q"], d["q"]]))
    assert K.counted["native"] == 1


def test_unfit_outputs_and_arrays_are_refused_before_anything_is_launched(K):
    """Prefill, schedule and the scheduled call, on both paths: what the kernel would write past or read as something else."""
    w = W.make_config("cfg3", num_seqs=3, ctx_scale=0.2)
    d = to_device(w)
    desc = K.attn_desc(d["q"], d["k"], d["tables"], max_context_len=w.max_context_len)
    ws, sched = K.new_workspace(desc), torch.empty(K.schedule_bytes(desc), dtype=torch.uint8, device="cuda")
    qs = torch.arange(4, dtype=torch.int32, device="cuda")
    q, out = d["q"], torch.empty_like(d["q"])
    prefill = dict(q=q, k_cache=d["k"], v_cache=d["v"], block_tables=d["tables"], context_lens=d["lens"], q_start=qs, scale=w.scale,
                   max_query_len=1, out=out)
    scheduled = dict(q=q, k_cache=d["k"], v_cache=d["v"], schedule=sched, scale=w.scale, out=out, desc=desc, workspace=ws)
    build = dict(block_tables=d["tables"], context_lens=d["lens"], desc=desc, schedule=sched)
    outs = [dict(out=x) for x in (out[:2], out[:, ::2], out.float(), out.half(), out.cpu())]
    cases = [(K.paged_attention_prefill, prefill, outs),
             (K.paged_attention_decode_scheduled, scheduled, outs + [dict(q=q[:2]), dict(v_cache=d["v"].float()), dict(workspace=ws.cpu())]),
             (K.attn_schedule_build, build, [dict(block_tables=d["tables"].long()), dict(context_lens=d["lens"].long()),
                                             dict(block_tables=d["tables"][:2]), dict(context_lens=d["lens"][:2]), dict(schedule=sched.cpu())])]
    for general in (False, True):
        if general:
            K.general()
        for call, ok, bad in cases:
            for b in bad:
                with pytest.raises((ValueError, TypeError)):
                    call(**{**ok, **b})
    assert K.counted["native"] == 0
