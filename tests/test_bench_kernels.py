"""bench.py names every kernel of the layer, and the key of its committed FFN
traffic covers every source an FFN launch is built from.  CPU only."""
import os
import re

import bench
from paper_2602_04870_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_04870_amd", "csrc")


def _function(text, name):
    body = text[text.index(f"mhlmoe_status {name}("):]
    return body[:body.index("\n}\n")]


def test_every_layer_kernel_is_reported():
    api = open(os.path.join(CSRC, "api.cpp")).read()
    for entry in ("run_cluster", "run_experts", "layer_impl", "backward_impl"):
        for kernel in re.findall(r'run_kernel\("(\w+)"', _function(api, entry)):
            assert kernel in bench.KERNELS, kernel
    # the per-step tables list the backward's kernels, too
    text = open(os.path.join(ROOT, "bench.py")).read()
    for table in re.findall(r'for kn in \(([^)]*"bwd_dw"[^)]*)\)', text):
        for kernel in ("bwd_dx", "bwd_combine", "dw_plan", "bwd_dw", "router_dw"):
            assert f'"{kernel}"' in table, (kernel, table)


def test_traffic_key_covers_the_ffn_sources():
    for name in build.SOURCES:
        text = open(os.path.join(CSRC, name)).read()
        if re.search(r"__global__[^;{]*\bffn_\w*kernel\(", text):
            assert name in bench.FFN_SOURCES, name
            for header in re.findall(r'#include "(\w+\.hpp)"', text):
                assert header in bench.FFN_SOURCES, (name, header)
