"""Lanes of a wave that hand values to each other through LDS.

The weight gradients' waves stage image rows in an LDS patch that other lanes of
the wave read, with no block barrier.  The hardware keeps a wave's LDS accesses
in order; the compiler has to be told, since per lane the store and the load are
of different addresses.  So in the kernels' optimised IR every turn from LDS
stores to loads and from loads to stores has a fence between, and so has the
store of an outer pixel, which may fall on another lane's row store in images
whose width is no multiple of the tile."""
import os
import re
import subprocess

import pytest

from paper_1906_11027_amd import build as B


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> lines of the device IR of the weight-gradient kernels"""
    if not os.path.exists(B.HIPCC):
        pytest.skip("no hipcc")
    ll = str(tmp_path_factory.mktemp("ir") / "nn.ll")
    subprocess.run([B.HIPCC] + [f for f in B.FLAGS if f != "-fPIC"] +
                   ["-x", "hip", "--cuda-device-only", "-emit-llvm", "-S", os.path.join(B.CSRC, "nn.hip"), "-o", ll],
                   check=True, capture_output=True, timeout=300)
    found, name = {}, None
    with open(ll) as f:
        for line in f:
            m = re.match(r"define .*amdgpu_kernel void @(\w*k_conv_bwd_w\w*)\(", line)
            if m:
                name = m.group(1)
                found[name] = []
            elif line.startswith("}"):
                name = None
            elif name:
                found[name].append(line.strip())
    return found


def _kind(line):
    """rows / pixel / load: an LDS access; fence; None: anything else"""
    if line.startswith("fence "):
        return "fence"
    if "addrspace(3)" not in line:
        return None
    if line.startswith("store "):
        return "rows" if line.startswith("store <4 x float>") else "pixel"
    return "load" if re.match(r"%\S+ = load ", line) else None


def _turns_without_fence(lines):
    """(before, after) access pairs of different kinds that some path joins with no fence between."""
    blocks, succ, label = {}, {}, "entry"
    for line in lines:
        m = re.match(r"([\w.$-]+):", line)
        if m:
            label = m.group(1)
        blocks.setdefault(label, [])
        if _kind(line):
            blocks[label].append((_kind(line), line))
        if re.match(r"(br|switch) |label %|i\d+ \S+, label", line):
            succ.setdefault(label, set()).update(re.findall(r"label %([\w.$-]+)", line))
    at_start, todo, bad = {"entry": set()}, ["entry"], set()
    while todo:                      # the last accesses that may reach a block
        label = todo.pop()
        last = set(at_start[label])
        for kind, line in blocks.get(label, []):
            if kind == "fence":
                last = set()
            else:
                bad |= {(was, line) for k, was in last if k != kind}
                last = {(kind, line)}
        for nxt in succ.get(label, ()):
            if nxt not in at_start or not last <= at_start[nxt]:
                at_start[nxt] = at_start.get(nxt, set()) | last
                todo.append(nxt)
    assert len(at_start) > len(blocks) // 2
    return sorted(bad)


def test_every_turn_has_a_fence(kernels):
    assert len(kernels) == 12   # three kinds of edge; 1, 2, 4 waves a row, and the 32 -> 32 kernel
    for name, lines in kernels.items():
        assert sum("addrspace(3)" in line for line in lines) > 20, name
        bad = _turns_without_fence(lines)
        assert not bad, "%s: %d turns, the first:\n%s\n%s" % (name, len(bad), *bad[0])
