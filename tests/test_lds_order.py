"""What the kernel sources must keep to where the compiler cannot check it:
LDS handed between the lanes of a wavefront, and LDS DMA that the compiler does
not track.  CPU only (reads the sources)."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_04870_amd", "csrc")


def _source(name):
    text = open(os.path.join(CSRC, name)).read()
    return re.sub(r"//[^\n]*", "", text)


def _block(text, head):
    """The brace block that follows head."""
    at = text.index("{", text.index(head))
    depth = 0
    for i in range(at, len(text)):
        depth += {"{": 1, "}": -1}.get(text[i], 0)
        if depth == 0:
            return text[at:i + 1]
    raise AssertionError(head)


def test_cross_lane_turns_order_their_lds_accesses():
    """Pieces that one lane writes and another reads: wave_lds_order() between
    the writes and the reads, and between the reads and the next writes."""
    for name, head in (("backward.hip", "void turn(RowFrag"), ("ffn_ws.hip", "auto turn_w =")):
        body = _block(_source(name), head)
        write = [m.start() for m in re.finditer(r"reinterpret_cast<u32x4\*>\(st\b", body)]
        read = [m.start() for m in re.finditer(r"reinterpret_cast<const u32x4\*>\(st\b", body)]
        order = [m.start() for m in re.finditer(r"wave_lds_order\(\)", body)]
        assert len(write) == 1 and len(read) == 1, name
        assert any(write[0] < o < read[0] for o in order), f"{name}: reads not after the writes"
        assert any(read[0] < o for o in order), f"{name}: next writes not after the reads"
    # the wavefront's tiles of the d_h-64 weight gradients: the same
    body = _block(_source("backward.hip"), "auto body = [&](Rows& q")
    assert body.count("wave_lds_order()") == 2


def test_untracked_lds_dma_is_not_mixed_with_tracked():
    """dma_lds16 writes m0 without the compiler's knowledge, so a kernel that
    issues it issues no tracked LDS DMA."""
    untracked = re.compile(r"\bdma_lds16\(|\bBwdDma<|\bdma\.issue\(")
    found = 0
    for name in sorted(os.listdir(CSRC)):
        if not name.endswith(".hip"):
            continue
        text = _source(name)
        for m in re.finditer(r"__global__[^{;]*?(\w+_kernel)\(", text):
            body = _block(text[m.start():], m.group(1) + "(")
            if untracked.search(body):
                found += 1
                assert "load_lds" not in body and "dma_buffer16" not in body, f"{name}: {m.group(1)}"
    assert found == 1  # bwd_dx_kernel
