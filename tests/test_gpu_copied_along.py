"""Requests that keep little: the workgroup that selects the rows copies them too (up to 64 KB of K and V per request and head)."""
import numpy as np
import pytest

from paper_2604_10235_amd import workloads as wl
from tests import parity_util as pu

pytestmark = pytest.mark.gpu


# Rows of 64, 128 and 256 bytes: one step of the workgroup and one row over, the limit and one row over (its own kernel), nothing but
# the window, everything; several requests, and workgroups of 256 to 1024 threads (few and many problems, short and long requests).
@pytest.mark.parametrize("d,kv", [(64, "fp8"), (64, "bf16"), (128, "bf16")])
@pytest.mark.parametrize("lens,budgets,heads", [([300, 40, 2000], [33, 32, 127], 4), ([300, 40, 2000], [128, 40, 65], 4), ([700, 129], [129, 128], 2),
                                                ([20000, 515], [257, 512], 3), ([20000, 600], [256, 513], 1), ([90, 40, 33], [64, 33, 32], 180)])
@pytest.mark.parametrize("select_mode", [0, 1])
def test_copied_rows(d, kv, lens, budgets, heads, select_mode):
    import torch
    from paper_2604_10235_amd import binding as b
    w = wl.scaled(wl.qwen7b_32k(), n_layers=1, n_q_heads=heads, n_kv_heads=heads, head_dim=d, window=32, seqlens=lens, budgets=budgets)
    q, k, v, prior = wl.make_all(w)
    if kv == "fp8":
        k, v = wl.bf16_bits_to_fp8_codes(k), wl.bf16_bits_to_fp8_codes(v)
    fused, steps = (b.DeviceProblem(w, q, k, v, prior, select_mode=select_mode) for _ in range(2))
    for x in (fused.k_out, fused.v_out):
        x.view(torch.uint8).fill_(0x5A)
    fused.compress()
    steps.score()
    steps.select()
    steps.gather()
    torch.cuda.synchronize()
    for name in ("scores", "idx", "k_out", "v_out"):
        assert torch.equal(getattr(fused, name).view(torch.uint8), getattr(steps, name).view(torch.uint8)), name
    idx = fused.idx.cpu().numpy()
    assert np.array_equal(b.DeviceProblem.bits(fused.k_out), pu.host_gather(k, idx, w.cu_seqlens(), w.cu_budgets()))
    assert np.array_equal(b.DeviceProblem.bits(fused.v_out), pu.host_gather(v, idx, w.cu_seqlens(), w.cu_budgets()))
