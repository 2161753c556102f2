"""GPU parity with the CPU oracle, bit for bit, at edges of the match searches and
of the passes in front of them: results at the first position of a batch order."""
import os

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2202_13951_amd import binding
from synth import channel, codes

pytestmark = pytest.mark.gpu
THREADS = min(16, os.cpu_count() or 1)


def _check(got, want, tag):
    cw, q, ab = (t.cpu().numpy() for t in got)
    bad = np.nonzero((cw != want[0]).any(axis=1) | (q.astype(np.uint64) != want[1]) | (ab != want[2]))[0]
    assert bad.size == 0, f"{tag}: {bad.size} differ, first {bad[:8].tolist()}: gpu {q[bad[:4]]} oracle {want[1][bad[:4]]}"


@pytest.mark.parametrize("n,m", [(64, 14), (127, 14), (300, 40)])
@pytest.mark.parametrize("budget", [1, 64, 6000])
def test_first_query_of_a_batch_order(gpu_device, n, m, budget):
    """A member that is the first pattern of the batch that the order puts first is
    query 1, and its flips are made (in the plain order query 1 flips nothing)."""
    print(f"first query of an order n={n} budget={budget}", flush=True)
    rng = np.random.default_rng(n)
    H = codes.rlc_H(n, n - m, seed=n)
    cw = channel.encode(codes.generator_matrix(H), rng.integers(0, 2, size=(64, n - m), dtype=np.uint8))
    pats = O.order_prefix_array(n, 4096)
    llr = np.empty((64, n), dtype=np.float32)
    order = np.empty((64, 64), dtype=np.uint8)
    for b in range(64):
        perm = rng.permutation(n)
        ranks = pats[64 * b]
        rx = cw[b].copy()
        rx[perm[ranks[ranks > 0] - 1]] ^= 1
        llr[b, perm] = (0.5 + 0.1 * np.arange(n)) * (2.0 * rx[perm] - 1)
        order[b] = np.concatenate([[b], rng.permutation(np.setdiff1d(np.arange(64), [b]))])
    got = binding.orbg_decode_ordered(H, torch.from_numpy(llr).to(gpu_device), budget,
                                      torch.from_numpy(order).to(gpu_device))
    want = O.decode_ordered(H, llr, budget, order, THREADS)
    assert (want[1] == 1).all() and (want[0] == cw).all()
    _check(got, want, f"order n={n} budget={budget}")
