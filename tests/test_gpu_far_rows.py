"""The d_h-128 kernels whose row buffers end at 4 GiB, on both sides of it
(2^24 (token, head) rows), against the CPU oracle: the expert FFN and the
layer backward at one slot per (token, head).  A few hundred tokens, at both
ends and on both sides of 2 GiB, choose among the first four experts and every
other token among the rest, so the oracle needs those tokens alone for their
outputs, their input gradients and the four experts' weight gradients."""
import numpy as np
import pytest
import torch

import paper_2602_04870_amd as mh
from tests.gpu_util import announce, check_expert_blocks, check_rows, needs_gpu, to_host_f64

pytestmark = [pytest.mark.gpu, needs_gpu]

NH, DH, NE, DFF = 8, 128, 16, 128
EDGE = (1 << 24) // NH  # tokens at which the rows reach 4 GiB


@pytest.mark.parametrize("expert", ["swiglu", "gelu"])
@pytest.mark.parametrize("T", [EDGE - 1, EDGE])
def test_rows_either_side_of_4_gib(T, expert, oracle_instance):
    announce(f"far rows {expert} T={T}")
    gen = torch.Generator(device="cuda").manual_seed(41)

    def normal(shape, std=1.0, dtype=torch.bfloat16):
        return (torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16) * std).to(dtype)

    X, dY = normal((T, NH, DH)), normal((T, NH, DH))
    W_router = normal((NH, NE, DH), DH ** -0.5, torch.float32)
    W1, W2 = normal((NH, NE, DFF, DH), DH ** -0.5), normal((NH, NE, DH, DFF), DFF ** -0.5)
    W3 = normal((NH, NE, DFF, DH), DH ** -0.5) if expert == "swiglu" else None
    idx = torch.randint(4, NE, (T, NH, 1), generator=gen, device="cuda", dtype=torch.int32)
    gate = 0.2 + 0.6 * torch.rand((T, NH, 1), generator=gen, device="cuda")
    rng = np.random.default_rng(43)
    rows = np.unique(np.concatenate([np.arange(64), T - 1 - np.arange(64),
                                     EDGE // 2 + np.arange(-32, 32), rng.integers(0, T, 64)]))
    r = torch.from_numpy(rows).cuda()
    idx[r] = torch.randint(0, 4, (len(rows), NH, 1), generator=gen, device="cuda",
                           dtype=torch.int32)

    def host(t):
        return None if t is None else to_host_f64(t)

    o_idx, o_gate = idx[r].cpu().numpy(), gate[r].cpu().numpy().astype(np.float64)
    args = (host(X[r]), o_idx, o_gate, host(W1))
    if expert == "swiglu":
        Y = mh.mhlmoe_experts(X, idx, gate, W1, W3, W2)
        want = oracle_instance.experts(*args, host(W3), host(W2))
    else:
        Y = mh.mhlmoe_experts_gelu(X, idx, gate, W1, W2)
        want = oracle_instance.experts_gelu(*args, host(W2))
    torch.cuda.synchronize()
    check_rows(to_host_f64(Y[r]), want, "bf16", f"far rows {expert} Y")
    del Y

    if expert == "swiglu":
        names = ("dX", "dW_router", "dW1", "dW3", "dW2")
        got = mh.mhlmoe_layer_backward(X, W_router, W1, W3, W2, idx, gate, dY)
    else:
        names = ("dX", "dW_router", "dW1", "dW2")
        got = mh.mhlmoe_layer_gelu_backward(X, W_router, W1, W2, idx, gate, dY)
    torch.cuda.synchronize()
    want = oracle_instance.layer_backward(host(X[r]), host(W_router), host(W1), host(W3), host(W2),
                                          o_idx, o_gate.astype(np.float32), host(dY[r]))
    counts = np.stack([np.bincount(o_idx[:, h].ravel(), minlength=4) for h in range(NH)])
    for n, g in zip(names, got):
        if n == "dX":
            check_rows(to_host_f64(g[r]), want[n], "bf16", f"far rows {expert} dX")
        else:
            check_expert_blocks(to_host_f64(g[:, :4].contiguous()), want[n][:, :4], counts,
                                f"far rows {expert} {n}")
