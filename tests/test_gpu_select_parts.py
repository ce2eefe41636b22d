"""Selection by parts (batches with a request beyond 65536 candidates) where its kernels branch: the request that a workgroup
finds one per lane (up to 64 of them) or by shares, and a list around the cut that a workgroup still holds in registers (16384
keys) or reads again, spread evenly, over the first or last parts alone, or ending on the edge of a part."""
import numpy as np
import pytest

from oracle import codecomp_oracle as orc
from tests.test_gpu_select_cases import W, crafted_rows, select_on_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("requests,long_at", [(1, 0), (2, 1), (63, 40), (64, 0), (64, 63), (65, 0), (65, 64)])
def test_a_long_request_among_some(requests, long_at):
    g = np.random.default_rng(100 * requests + long_at)
    lens = [int(x) + W for x in g.integers(0, 20000 if requests < 4 else 900, size=requests)]
    lens[long_at] = 8192 * 8 + 5 + W
    needs = [int(g.integers(0, n - W + 1)) for n in lens]
    needs[long_at] = 7000
    rows = np.concatenate([crafted_rows(n - W, max(1, b), seed=i)[[3, 4, 6, 11]] if n > W else np.zeros((4, W), np.float32)
                           for i, (n, b) in enumerate(zip(lens, needs))], axis=1)
    idx, cu, cb = select_on_device(rows, lens, [b + W for b in needs])
    assert np.array_equal(idx.astype(np.int64), orc.select_packed(rows.astype(np.float64)[None], cu, cb, W))


@pytest.mark.parametrize("listed", [1, 63, 64, 8192, 16383, 16384, 16385, 24576, 60000])
def test_lists_of_a_length(listed):
    npre, n = 100_003, 100_003 + W
    g = np.random.default_rng(listed)
    rows = []
    for where in (g.choice(npre, size=listed, replace=False), np.arange(listed), np.arange(npre - listed, npre),
                  (np.arange(listed) + 8192 * 3) % npre, 8192 * 11 - 1 - np.arange(listed)):
        r = g.uniform(0.1, 0.2, n).astype(np.float32)
        r[where] = 1.0 + 2.0 ** -12 * g.integers(0, 5, size=listed).astype(np.float32)       # one bin, five values
        rows.append(r)
    rows = np.stack(rows)
    for need in {1, (listed + 1) // 2, listed}:
        idx, cu, cb = select_on_device(rows, [n], [need + W])
        assert np.array_equal(idx[0].astype(np.int64), orc.select(rows.astype(np.float64), W, need + W)), need
