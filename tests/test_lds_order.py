"""Kernels that refill LDS slots behind a barrier: in the code built from their
sources no wave passes a barrier with an LDS read of its own still in flight
(another wave's next load could land in the slot being read)."""
import importlib.util
import os
import re
import subprocess

import pytest

PKG = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2608_13426_amd")
_spec = importlib.util.spec_from_file_location("_rmm_build_script", os.path.join(PKG, "build.py"))
build = importlib.util.module_from_spec(_spec)
_spec.loader.exec_module(build)


def _blocks(lines):
    """{label: (instructions, successors)} of one function's assembly."""
    blocks, name, cur = {}, "entry", []
    order = ["entry"]
    blocks[name] = cur
    for ln in lines:
        m = re.match(r"(\.LBB\w+):", ln)
        if m:
            name, cur = m.group(1), []
            blocks[name] = cur
            order.append(name)
        elif re.match(r"\s+[a-z]", ln):
            cur.append(ln.split(";")[0].strip())
    out = {}
    for i, b in enumerate(order):
        succ, falls = set(), True
        for ins in blocks[b]:
            op = ins.split()[0]
            if op.startswith("s_cbranch") or op == "s_branch":
                succ.add(ins.split()[1])
            if op in ("s_branch", "s_endpgm"):
                falls = False
        if falls and i + 1 < len(order):
            succ.add(order[i + 1])
        out[b] = (blocks[b], succ)
    return out


def reads_in_flight(lines):
    """Per s_barrier of one function: the most LDS reads that can be in flight.

    LDS operations of a wave finish in order, so after a wait for lgkmcnt(n)
    at most the last n of them are pending (scalar loads share the counter,
    which only lowers that number)."""
    blocks = _blocks(lines)
    state = {b: None for b in blocks}
    state["entry"] = ()
    work, worst = ["entry"], {}
    while work:
        b = work.pop()
        pend = list(state[b])
        for n, ins in enumerate(blocks[b][0]):
            op = ins.split()[0]
            if op.startswith("ds_"):
                pend = (pend + [op.startswith("ds_read")])[-64:]
            elif op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", ins)
                if m:
                    pend = pend[len(pend) - min(int(m.group(1)), len(pend)):]
            elif op == "s_barrier":
                worst[b, n] = max(worst.get((b, n), 0), sum(pend))
        for s in blocks[b][1]:
            old = state[s]
            if old is None:
                new = tuple(pend)
            else:                                   # newest last: align at the end
                size = max(len(old), len(pend))
                a, c = [False] * (size - len(old)) + list(old), [False] * (size - len(pend)) + pend
                new = tuple(x or y for x, y in zip(a, c))
            if new != old:
                state[s] = new
                work.append(s)
    return list(worst.values())


def test_pending_reads_are_found():
    """The count on hand-written loops, with the read's wait before and after the barrier."""
    loop = ["f:", ".LBB0_1:", "\tds_read_b64_tr_b16 v[0:1], v2", "\tds_read_b128 v[4:7], v3",
            "\ts_waitcnt lgkmcnt(1)", "\ts_barrier", "\ts_waitcnt lgkmcnt(0)", "\ts_cbranch_scc1 .LBB0_1",
            "\ts_barrier", "\ts_endpgm"]
    assert reads_in_flight(loop) == [1, 0]
    loop[4], loop[6] = loop[6], loop[4]
    assert reads_in_flight(loop) == [0, 0]
    carried = ["f:", ".LBB0_1:", "\ts_barrier", "\ts_waitcnt lgkmcnt(0)", "\tds_write_b32 v0, v1",
               "\tds_read_b32 v0, v1", "\ts_cbranch_scc1 .LBB0_1", "\ts_endpgm"]
    assert reads_in_flight(carried) == [1]


@pytest.mark.parametrize("source", ["gemm.hip", "gemm_mid.hip", "gemv_shared.hip", "attn.hip", "attn_few.hip", "qk.hip"])
def test_no_lds_read_in_flight_at_a_barrier(source, tmp_path):
    asm = tmp_path / "out.s"
    subprocess.run([build.HIPCC, *build.CFLAGS, "-S", "--cuda-device-only", os.path.join(build.CSRC, source),
                    "-o", str(asm)], check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    seen, kernel, lines = 0, None, []
    for ln in asm.read_text().splitlines():
        m = re.match(r"(_Z\w+):", ln)
        if m:
            kernel, lines = m.group(1), []
        elif ln.startswith(".Lfunc_end") and kernel:
            counts = reads_in_flight(lines)
            seen += len(counts)
            assert not any(counts), (kernel, counts)
            kernel = None
        elif kernel:
            lines.append(ln)
    assert seen > 0
