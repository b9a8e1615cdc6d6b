"""The native call path on CPU tensors: kvc_call.cpp compiled with CPU tensors taken for device tensors and bound to
functions that only record that they were called."""
import os
import subprocess
import sys
import textwrap

import pytest

import paper_2503_13773_amd.build as B

SETUP = """
import ctypes, importlib.machinery, importlib.util, sys, warnings
import torch
from paper_2503_13773_amd.binding import AttnDesc
warnings.simplefilter("ignore")
loader = importlib.machinery.ExtensionFileLoader("kvc_call", sys.argv[1])
C = importlib.util.module_from_spec(importlib.util.spec_from_loader("kvc_call", loader))
loader.exec_module(C)
vp, sz, f, i32, i64 = ctypes.c_void_p, ctypes.c_size_t, ctypes.c_float, ctypes.c_int32, ctypes.c_int64
called = []
def stub(name, result, *types):
    def record(*args):
        called.append(name)
        return 0
    return ctypes.CFUNCTYPE(result, *types)(record)
stubs = [stub("decode", i32, *[vp] * 5, f, vp, vp, vp, sz, vp), stub("bytes", sz, vp),
         stub("scheduled", i32, *[vp] * 4, sz, f, vp, vp, vp, sz, vp), stub("build", i32, vp, vp, vp, vp, sz, vp),
         stub("prefill", i32, *[vp] * 6, f, vp, vp, i32, i32, vp), stub("append", i32, *[vp] * 8),
         stub("copy", i32, vp, vp, vp, i64, vp)]
C.bind(*(ctypes.cast(s, vp).value for s in stubs), AttnDesc)
bf = torch.bfloat16
q, k = torch.zeros(3, 8, 64, dtype=bf), torch.zeros(5, 2, 16, 64, dtype=bf)
bt, cl, qs = torch.zeros(3, 4, dtype=torch.int32), torch.zeros(3, dtype=torch.int32), torch.arange(4, dtype=torch.int32)
new, ws, sched = torch.zeros(3, 2, 64, dtype=bf), torch.zeros(4096, dtype=torch.uint8), torch.zeros(512, dtype=torch.uint8)
pool, pairs = torch.zeros(2, 4, 32, dtype=bf), torch.zeros(1, 2, dtype=torch.int64)
desc = AttnDesc(3, 8, 2, 64, 16, 4, 5, 1, 0, 0, 0, 0)
good = {"decode": [q, k, k, bt, cl, 0.1, q.clone(), desc, ws, 0],
        "scheduled": [q, k, k, sched, 0.1, q.clone(), desc, ws, 0],
        "schedule_build": [bt, cl, desc, sched, 0],
        "prefill": [q, k, k, bt, cl, qs, 0.1, 1, q.clone(), 0, 0],
        "append": [new, new, k, k, bt, cl, 0],
        "block_copy": [pool, pool, pairs, 0]}
def call(name, **change):
    args = list(good[name])
    for at, value in change.items():
        args[int(at[1:])] = value
    called.clear()
    rc = getattr(C, name)(*args)
    assert rc == (0 if called else None), (name, rc, called)   # None: the library has not been called
    return bool(called)
for name in good:
    assert call(name), name
"""


@pytest.fixture(scope="module")
def module(tmp_path_factory):
    folder = tmp_path_factory.mktemp("kvc_call")
    text = open(os.path.join(B.CSRC, "kvc_call.cpp")).read()
    assert "is_cuda()" in text
    source = folder / "kvc_call_cpu.cpp"
    source.write_text(text.replace("is_cuda()", "is_cpu()"))
    return B.build_call_module(source=str(source), out=str(folder / "kvc_call.so"))


def run(module, body):
    r = subprocess.run([sys.executable, "-c", SETUP + textwrap.dedent(body), module], cwd=B.ROOT, capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stderr[-2000:])


def test_a_nested_tensor_is_left_to_the_general_path(module):
    # exactly a torch.Tensor, strided, contiguous and with storage, but sizes() throws
    run(module, """
        nested = {bf: torch.nested.nested_tensor([torch.zeros(8, 64, dtype=bf), torch.zeros(4, 64, dtype=bf)]),
                  torch.int32: torch.nested.nested_tensor([torch.zeros(4, dtype=torch.int32)] * 3),
                  torch.uint8: torch.nested.nested_tensor([torch.zeros(4096, dtype=torch.uint8)]),
                  torch.int64: torch.nested.nested_tensor([torch.zeros(2, dtype=torch.int64)])}
        assert type(nested[bf]) is torch.Tensor and nested[bf].is_contiguous() and nested[bf].layout == torch.strided
        for name, args in good.items():
            for i, a in enumerate(args):
                if isinstance(a, torch.Tensor):
                    assert not call(name, **{f"a{i}": nested[a.dtype]}), (name, i)
    """)


def test_only_a_descriptor_is_read_as_one(module):
    # 48 bytes of anything else: the general path's ctypes call refuses them
    run(module, """
        class Other(ctypes.Structure):
            _fields_ = AttnDesc._fields_
        class Derived(AttnDesc):
            pass
        words = [getattr(desc, f) for f, _ in AttnDesc._fields_]
        for name, at in (("decode", "a7"), ("scheduled", "a6"), ("schedule_build", "a2")):
            for what in (bytes(desc), bytearray(bytes(desc)), Other(*words)):
                assert not call(name, **{at: what}), (name, type(what))
            assert call(name, **{at: Derived(*words)})
    """)


def test_what_the_kernel_would_write_or_read_out_of_range_is_not_taken(module):
    run(module, """
        small, wide, strided = q[:2], q.float(), torch.zeros(3, 8, 128, dtype=bf)[..., ::2]
        meta = torch.zeros(3, 8, 64, dtype=bf, device="meta")
        for out in (small, wide, strided, meta, q.half()):
            for name, at in (("prefill", "a8"), ("scheduled", "a5"), ("decode", "a5")):
                assert not call(name, **{at: out}), (name, out.shape, out.dtype)
        for flat in (torch.zeros(3 * 8 * 64, dtype=bf), torch.zeros(4, 8, 64, dtype=bf)):   # as large as q or larger
            assert call("prefill", a8=flat) and call("scheduled", a5=flat)
        assert not call("scheduled", a0=small) and not call("scheduled", a0=strided)
        assert not call("scheduled", a1=k[:4]) and not call("scheduled", a2=k.float())
        for at, what in (("a0", bt.long()), ("a1", cl.long()), ("a0", bt[:2]), ("a1", cl[:2]), ("a0", bt.t())):
            assert not call("schedule_build", **{at: what}), (at, what.shape, what.dtype)
        for name, at in (("decode", "a8"), ("scheduled", "a7"), ("scheduled", "a3"), ("schedule_build", "a3")):
            assert not call(name, **{at: torch.zeros(4096, dtype=torch.uint8, device="meta")}), (name, at)
    """)
