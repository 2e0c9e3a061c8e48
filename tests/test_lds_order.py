"""Order of LDS reads and refills in the kernels whose workgroup halves take turns (CPU only).

Their barriers are bare s_barriers, which wait for nothing, so that transfers into LDS stay in
flight across them. An LDS read must then be waited for before the barrier after which another
wave may refill its buffer. In these kernels every fragment is read in one half phase and used
by the MFMAs of the next, and no buffer is refilled sooner than one barrier after those: so a
wave's LDS reads may be in flight across one barrier, never across two. The check walks the
device assembly that the library's own flags give, over every path of each kernel."""
import os
import re
import subprocess

import pytest

from paper_2608_15171_amd import build as B

MAX_AGE = 4


def _kernels(tmp_path, source):
    out = tmp_path / (source + ".s")
    cmd = [B.hipcc(), *[f for f in B.HIPCC_FLAGS if f != "-shared"], "--cuda-device-only", "-S", "-I", B.INCLUDE,
           "-I", B.CSRC, os.path.join(B.CSRC, source), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    bodies, name = {}, None
    for line in out.read_text().splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            name = m.group(1)
            bodies[name] = []
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name:
            line = line.split(";")[0].strip()
            if line and (not line.startswith(".") or line.endswith(":")):
                bodies[name].append(line)
    return bodies


def _blocks(body):
    """Basic blocks: a list of (instructions, successor block numbers)."""
    blocks, labels, cur = [], {}, []
    for line in body:
        if line.endswith(":"):
            if cur:
                blocks.append(cur)
                cur = []
            labels[line[:-1]] = len(blocks)
            continue
        cur.append(line)
        if line.split()[0].startswith(("s_cbranch", "s_branch", "s_endpgm")):
            blocks.append(cur)
            cur = []
    if cur:
        blocks.append(cur)
    out = []
    for i, b in enumerate(blocks):
        op = b[-1].split()
        assert not op[0].startswith(("s_setpc", "s_call", "s_swappc")), b[-1]
        nxt = [i + 1] if i + 1 < len(blocks) else []
        if op[0] == "s_endpgm":
            nxt = []
        elif op[0] == "s_branch":
            nxt = [labels[op[1]]]
        elif op[0].startswith("s_cbranch"):
            nxt = nxt + [labels[op[1]]]
        out.append((b, nxt))
    return out


def longest_flight(body):
    """The most barriers that an LDS read can be in flight across, and where. A state is the
    ages (barriers crossed) of the LDS operations in flight, oldest first; they complete in
    order, so a wait for lgkmcnt(n) leaves the youngest n. (Scalar loads count in lgkmcnt too:
    then fewer than n of the LDS operations are left.)"""
    blocks = _blocks(body)
    start = {0: ()}
    todo, worst, where = [0], 0, ""
    while todo:
        i = todo.pop()
        ages = list(start[i])
        for line in blocks[i][0]:
            op = line.split()[0]
            if op.startswith("ds_"):
                ages.append(0)
            elif op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", line)
                if m:
                    ages = ages[len(ages) - min(len(ages), int(m.group(1))):]
            elif op == "s_barrier":
                ages = [min(a + 1, MAX_AGE) for a in ages]
                if ages and max(ages) > worst:
                    worst, where = max(ages), f"block {i}: {len(ages)} reads in flight"
        for n in blocks[i][1]:
            old = start.get(n)
            new = tuple(ages)
            if old is not None:          # paths meet: the older of each pair, counted from the youngest
                k = max(len(old), len(new))
                a, b = (0,) * (k - len(old)) + old, (0,) * (k - len(new)) + new
                new = tuple(max(x, y) for x, y in zip(a, b))
            new = new[-64:]
            if new != old:
                start[n] = new
                todo.append(n)
    return worst, where


@pytest.mark.parametrize("text,want", [
    # waited for by the MFMAs after the next barrier
    (["ds_read_b128 v[0:3], v9", "s_barrier", "s_waitcnt lgkmcnt(0)", "s_barrier", "s_endpgm"], 1),
    # the first of two reads is left to a wait for the second alone
    (["ds_read_b128 v[0:3], v9", "ds_read_b128 v[4:7], v9", "s_barrier", "s_waitcnt lgkmcnt(1)", "s_barrier",
      "s_endpgm"], 2),
    # round a loop, where only the back edge carries the read
    ([".LBB0_1:", "s_barrier", "s_waitcnt vmcnt(3)", "s_barrier", "s_waitcnt lgkmcnt(0)", "ds_read_b128 v[0:3], v9",
      "s_cbranch_scc1 .LBB0_1", "s_endpgm"], 2)])
def test_the_walk_counts_barriers(text, want):
    assert longest_flight(text)[0] == want


@pytest.mark.parametrize("source,kernels", [("gateup.hip", ["gateup_kernelILi256ELb0E", "gateup_kernelILi256ELb1E",
                                                            "gateup_kernelILi128ELb0E", "gateup_kernelILi128ELb1E"]),
                                            ("attn_step.hip", ["attn_step_kernelILi8E"])])
def test_no_lds_read_is_in_flight_across_two_barriers(tmp_path, source, kernels):
    bodies = _kernels(tmp_path, source)
    for k in kernels:
        name, = [n for n in bodies if k in n]
        assert sum(l.startswith("s_barrier") for l in bodies[name]) >= 4 and \
            sum(l.startswith("ds_read") for l in bodies[name]) >= 16, name
        worst, where = longest_flight(bodies[name])
        assert worst <= 1, f"{name}: an LDS read in flight across {worst} barriers ({where})"
