"""The host side of the dispatch rules in csrc/launch.hpp, built with g++
(tests/dispatch_rules_check.cpp).  CPU only."""
import os
import shutil
import subprocess

import pytest

import paper_2602_04870_amd as mh

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_04870_amd", "csrc")


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    exe = str(tmp_path_factory.mktemp("rules") / "dispatch_rules_check")
    cmd = [gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{CSRC}",
           "-Wno-attributes", os.path.join(ROOT, "tests", "dispatch_rules_check.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-4000:]
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, (res.stdout + res.stderr)[-4000:]
    return [ln.split() for ln in res.stdout.splitlines()]


def test_weight_gradients_take_two_chunks_at_every_batch(lines):
    """An even number of d_ff chunks goes two per workgroup whatever the batch;
    past a 4 GiB row buffer by 64-bit addresses."""
    rows = [[int(v) for v in ln[1:]] for ln in lines if ln[0] == "dw"]
    assert len(rows) == 16 * 3 * 7
    one, two, two_far = 0, 1, 2
    for T, Nh, dff, form in rows:
        if dff % 64:
            assert form == one
        else:
            assert form == (two if T * Nh * 256 < 1 << 32 else two_far)


def test_stationary_ffn_shares_are_equal_in_cost(lines):
    """The cut of the weight-stationary FFN's tile list: complete and in order,
    and no share dearer than an equal one by more than a tile and the weights
    it starts and ends with."""
    rows = [ln for ln in lines if ln[0] == "shares"]
    assert len(rows) == 14
    for _, what, ntot, nexp, sw, bad, equal, dearest in rows:
        assert bad == "0", what
        assert int(dearest) <= float(equal) + 1 + 2 * int(sw), (what, equal, dearest)


@pytest.mark.parametrize("shape,layer,backward", [
    ((256, 4, 64, 16, 2, 128, mh.MHLMOE_F32), 552960, None),
    ((4096, 8, 128, 64, 8, 256, mh.MHLMOE_BF16), 70433792, 70831360),
    ((16384, 16, 128, 128, 8, 256, mh.MHLMOE_BF16), 564454400, 566568192),
    ((16384, 16, 128, 256, 16, 128, mh.MHLMOE_BF16), None, 1133135104),
    ((8192, 8, 128, 768, 8, 128, mh.MHLMOE_BF16), 143893504, 147350784),
    ((3001, 5, 64, 100, 5, 96, mh.MHLMOE_BF16), 10624768, 10775808)])
def test_workspace_of_calls_without_the_stationary_ffn(shape, layer, backward):
    """Workspace sizes as they were before that kernel's longer tile lists
    (None: a forward that takes it, or no backward in fp32)."""
    for op, want in ((mh.MHLMOE_OP_LAYER, layer), (mh.MHLMOE_OP_LAYER_BACKWARD, backward)):
        if want is not None:
            assert mh.mhlmoe_workspace_size(op, *shape) == want
