"""The layer kernel's copy pipeline as compiled: a wavefront waits for its
asynchronous copies by counting the vector loads issued after them, so the
loads have to stay where the source issues them."""
import os
import re
import subprocess

import pytest

from paper_2512_08557_amd import build as B


def _assembly(tmp_path, shapes):
    src = os.path.join(B.CSRC, "layer.hip")
    out = str(tmp_path / "layer.s")
    table = "-DSSC_ALL_SHAPES(X)=" + " ".join(f"X({a},{b},{s})" for a, b, s in shapes)
    r = subprocess.run([B.HIPCC, *B.COMMON, table, "--cuda-device-only", "-S", src, "-o", out], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr
    with open(out) as f:
        return f.read()


def _kernels(text):
    for m in re.finditer(r"^(_ZN3ssc12layer_kernel\w+):.*?^\s+s_endpgm", text, re.S | re.M):
        yield m.group(1), m.group(0)


def _blocks(body):
    """Basic blocks: split at labels and after branches."""
    cur = []
    for line in body.splitlines():
        ins = line.strip()
        if re.match(r"^\.LBB\w+:", ins):
            yield cur
            cur = []
        elif re.match(r"^[a-z]", ins):
            cur.append(ins)
            if ins.startswith(("s_cbranch", "s_branch", "s_setpc")):
                yield cur
                cur = []
    yield cur


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="needs the HIP compiler")
def test_weights_are_loaded_ahead_of_a_conditional_unit(tmp_path):
    """128 input channels: 36 units over 8 wavefronts, so four of them have one
    unit more, in a branch.  Its weights are issued with the copies of their
    unit, not inside the branch behind the last wait."""
    n = 0
    for name, body in _kernels(_assembly(tmp_path, [(128, 8, 1), (128, 32, 1), (128, 128, 1), (128, 64, 2)])):
        n += 1
        for blk in _blocks(body):
            has = {k: any(i.startswith(k) for i in blk)
                   for k in ("ds_read_b128", "v_mfma", "global_load_dwordx4", "global_load_lds")}
            if has["ds_read_b128"] and has["v_mfma"] and has["global_load_dwordx4"]:
                assert has["global_load_lds"], f"{name}: weights loaded where they are used"
    assert n == 24


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="needs the HIP compiler")
def test_the_kernels_fit_their_registers(tmp_path):
    """Eight wavefronts of a workgroup share a compute unit's registers, 256 each;
    what does not fit goes to scratch memory in every tile.  fp32 kernels of
    sparse backbones hold the most (lists, active-set words, three planes): at
    most 8 registers spill, and no other kernel's."""
    text = _assembly(tmp_path, [(32, 64, 1), (64, 64, 1), (64, 128, 2), (128, 128, 1), (256, 256, 1)])
    n = 0
    for blk in re.split(r"\n  - \.agpr_count", text)[1:]:
        name = re.search(r"\.name:\s+(\S+)", blk).group(1)
        m = re.search(r"layer_kernelILi(\d+)ELi(\d+)ELi(\d)ELb(\d)ELb(\d)ELb(\d)", name)
        if not m:
            continue
        n += 1
        spill = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", blk).group(1))
        assert spill <= (8 if m.group(4) == "0" and m.group(6) == "1" else 0), f"{name}: {spill} registers"
    assert n == 30


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="needs the HIP compiler")
def test_the_copy_pipeline_is_not_drained(tmp_path):
    """256 input channels on dense handles: nine units a wavefront, the copies of
    three in flight.  Between the first matrix instruction of a tile and its last copy no wait is
    for everything; the compiler adds such waits where the source waits for less
    than a unit's weights need."""
    n = 0
    for name, body in _kernels(_assembly(tmp_path, [(256, 256, 1), (256, 64, 2)])):
        if not re.search(r"ELb[01]ELb0ELb0E", name):     # sparse kernels wait for their counters
            continue
        lines = [x.strip() for x in body.splitlines()]
        copies = [k for k, x in enumerate(lines) if x.startswith("global_load_lds")]
        # tiles: runs of copies; the plan and the epilogues have none
        units = 0
        k = copies[0]
        while k <= copies[-1]:
            if lines[k].startswith("s_barrier"):
                units = 0
            units += lines[k].startswith("v_mfma")
            if units and any(c > k for c in copies) and re.match(r"s_waitcnt.*vmcnt\(0\)", lines[k]):
                nxt = next(c for c in copies if c > k)
                between = any(x.startswith("s_barrier") for x in lines[k:nxt])
                assert between, f"{name}: line {k} waits for every load in flight"
            k += 1
        n += 1
    assert n == 4
