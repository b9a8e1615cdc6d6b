"""What the compiler made of the balanced decode kernels' publication protocols (no GPU needed).

A cut row's partial travels from one wavefront to another inside a launch: the writer stores
it with device-scope accesses, waits until those stores have completed and only then adds to
the row's counter word; the reader fetches the slot once the counter shows the publication.
The wait is an explicit instruction in the source because a release fence at workgroup scope
compiles to no wait at all on gfx950.  This test compiles the kernel to assembly with the
library's own flags and checks that the wait is there in every instance of the kernel, so that
a compiler or source change that drops it is seen on the CPU and not as a rare wrong result.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2503_13773_amd import build as B

SRC = os.path.join(B.CSRC, "paged_attention_mfma_stream.hip")


def _assembly(tmp_path, src=SRC):
    hipcc = B._hipcc()
    if not (shutil.which(hipcc) or os.path.exists(hipcc)):
        pytest.skip("hipcc not available")
    out = tmp_path / "stream.s"
    flags = [f for f in B.FLAGS if f != "-fPIC"]
    r = subprocess.run([hipcc, *flags, "--cuda-device-only", "-S", src, "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return out.read_text().splitlines()


def test_partial_stores_complete_before_the_publication(tmp_path):
    lines = _assembly(tmp_path)
    kernels, name = {}, None
    for ln in lines:
        m = re.match(r"^(_ZN\S*pa_stream_mfma_kernel\S*):", ln)
        if m:
            name = m.group(1)
            kernels[name] = []
        elif name is not None:
            kernels[name].append(ln.strip())
            if ln.strip().startswith("s_endpgm"):
                name = None
    assert len(kernels) >= 4, sorted(kernels)
    checked = 0
    for name, body in kernels.items():
        # publications are the counter adds whose result is not read back (no sc0 on the add)
        pubs = [i for i, ln in enumerate(body) if ln.startswith("global_atomic_add") and "sc0" not in ln]
        stores = [i for i, ln in enumerate(body) if ln.startswith("buffer_store_dword") and "sc1" in ln]
        if not stores:      # the schedule-building instance streams nothing and publishes nothing
            assert not pubs, name
            continue
        assert pubs, name
        for i in pubs:
            before = [j for j in stores if j < i]
            assert before, (name, body[i])
            between = body[before[-1] + 1:i]
            assert any(re.match(r"s_waitcnt\b.*vmcnt\(0\)", ln) for ln in between), \
                f"{name}: no wait for the partial's stores before `{body[i]}`"
            checked += 1
    assert checked >= 4


def test_pieces_are_published_before_they_are_counted(tmp_path):
    """The kernel of few rows: every wavefront of a workgroup waits for its own stores of the piece, then all meet at a
    barrier, then one lane counts the piece at the row's counter (an add whose result it reads)."""
    kernels, name = {}, None
    for ln in _assembly(tmp_path, os.path.join(B.CSRC, "paged_attention_mfma_rows.hip")):
        m = re.match(r"^(_ZN\S*pa_rows_mfma_kernel\S*):", ln)
        if m:
            name = m.group(1)
            kernels[name] = []
        elif ln.startswith(".Lfunc_end"):
            name = None
        elif name is not None:
            kernels[name].append(ln.strip())
    checked = 0
    for name, body in kernels.items():
        adds = [i for i, ln in enumerate(body) if ln.startswith("global_atomic_add")]
        stores = [i for i, ln in enumerate(body) if ln.startswith("buffer_store_dword") and "sc1" in ln]
        assert bool(adds) == bool(stores), name             # the schedule-building instance has neither
        for i in adds:
            before = [j for j in stores if j < i]
            assert before and not [j for j in stores if j > i], (name, body[i])
            between = body[before[-1] + 1:i]
            waits = [j for j, ln in enumerate(between) if re.match(r"s_waitcnt\b.*vmcnt\(0\)", ln)]
            assert waits, f"{name}: no wait for the piece's stores before `{body[i]}`"
            assert any(ln.startswith("s_barrier") for ln in between[waits[0]:]), \
                f"{name}: no barrier between the wait for the piece's stores and `{body[i]}`"
            checked += 1
    assert checked >= 3, sorted(kernels)


def test_partitions_are_published_before_they_are_counted(tmp_path):
    """The vector-ALU kernel where the last partition of a row merges it: as in the kernel of few rows."""
    kernels, name = {}, None
    for ln in _assembly(tmp_path, os.path.join(B.CSRC, "paged_attention_valu.hip")):
        m = re.match(r"^(_ZN\S*pa_partial_valu_kernel\S*):", ln)
        if m:
            name = m.group(1)
            kernels[name] = []
        elif ln.startswith(".Lfunc_end"):
            name = None
        elif name is not None:
            kernels[name].append(ln.strip())
    checked = 0
    for name, body in kernels.items():
        adds = [i for i, ln in enumerate(body) if ln.startswith("global_atomic_add")]
        for i in adds:
            before = [j for j in range(i) if body[j].startswith("global_store") and "sc1" in body[j]]
            assert len(before) >= 2, name                   # accumulator, and maximum and sum
            between = body[before[-1] + 1:i]
            waits = [j for j, ln in enumerate(between) if re.match(r"s_waitcnt\b.*vmcnt\(0\)", ln)]
            assert waits, f"{name}: no wait for the partition's stores before `{body[i]}`"
            assert any(ln.startswith("s_barrier") for ln in between[waits[0]:]), \
                f"{name}: no barrier between the wait for the partition's stores and `{body[i]}`"
            checked += 1
    assert checked >= 16, sorted(kernels)


def test_score_products_of_the_wide_prefill_need_no_wait_states(tmp_path):
    """The wide prefill kernel's score products are inline asm, for which the compiler inserts no wait states: operands
    must not come from a vector instruction one or two before, and the scores of a product must not be touched by a
    vector instruction until two more matrix instructions (8 passes each, 11 states are needed) have been issued."""
    def registers(operand):
        m = re.match(r"^([va])\[(\d+):(\d+)\]$", operand) or re.match(r"^([va])(\d+)$", operand)
        if not m:
            return set()
        return {(m.group(1), i) for i in range(int(m.group(2)), int(m.group(m.lastindex)) + 1)}

    products, kernel = 0, False
    recent, pending = [], {}      # the last instructions' results; registers of scores -> matrix instructions since
    for ln in _assembly(tmp_path, os.path.join(B.CSRC, "paged_attention_prefill_wide.hip")):
        if re.match(r"^_ZN\S*pa_prefill_wide_kernel\S*:", ln):
            kernel, recent, pending = True, [], {}
        t = ln.strip()
        if not kernel or not t or t[0] in ".;_":
            continue
        if t.startswith("s_endpgm"):
            kernel = False
            continue
        op, _, rest = t.partition(" ")
        operands = [o.strip() for o in rest.split(";")[0].split(",")]
        touched = set().union(*map(registers, operands)) if operands else set()
        if op.startswith("v_mfma_f32_32x32x16"):
            pending = {r: n + 1 for r, n in pending.items() if n < 2}
            if operands[0].startswith("v"):
                products += 1
                sources = registers(operands[1]) | registers(operands[2])
                assert not sources & set().union(*recent[-2:], set()), f"operand written just before `{t}`"
                pending.update({r: 0 for r in registers(operands[0])})
            recent.append(set())
        elif op.startswith("v_"):
            early = [r for r in touched if pending.get(r, 2) < 2]
            assert not early, f"`{t}` touches a score right behind its product"
            recent.append(registers(operands[0]))
        elif op != "s_waitcnt":
            recent.append(set())
    assert products >= 2 * 6 * 16, products    # four unrolled turns and two loops of single ones, in two instances
