"""GPU parity of the match search and its first pass (match_impl.h, first_impl.h)
against the CPU oracle, bit for bit, where they can go wrong: the fewest check
bits, every keys-per-lane width with ragged lengths, dependent columns among
the least reliable ranks, tied magnitudes, budgets around the first batch and
the reordered prefix, both sides of the one-launch batch size."""
import os

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2202_13951_amd import binding
from synth import channel, codes

pytestmark = pytest.mark.gpu
THREADS = min(16, os.cpu_count() or 1)
DIRECT = 24576                       # largest batch decoded by one launch


def _check(got, want, tag):
    cw, q, ab = (t.cpu().numpy() for t in got)
    bad = np.nonzero((cw != want[0]).any(axis=1) | (q.astype(np.uint64) != want[1]) | (ab != want[2]))[0]
    assert bad.size == 0, f"{tag}: {bad.size} differ, first {bad[:8].tolist()}: gpu {q[bad[:4]]} oracle {want[1][bad[:4]]}"


@pytest.mark.parametrize("n,m,blocks,ebn0,budget", [
    (9, 1, 50, 2.0, 512), (13, 3, 70, 1.0, 8192), (60, 6, 33000, 3.0, 5000), (120, 8, 70000, 4.0, 3000),
    (11, 10, 400, 2.0, 2048), (12, 10, DIRECT + 9, 3.0, 4096), (40, 10, DIRECT + 1, 4.0, 3000),
    (64, 33, DIRECT + 63, 4.0, 300), (65, 11, DIRECT, 4.0, 2000), (128, 64, DIRECT + 7, 4.0, 100),
    (129, 24, DIRECT + 5, 4.5, 700), (257, 20, DIRECT + 1, 5.5, 1000), (513, 22, DIRECT + 3, 6.0, 300),
    (1024, 40, 300, 5.5, 20000)])
def test_widths_and_batch_sizes(gpu_device, n, m, blocks, ebn0, budget):
    print(f"match n={n} m={m} blocks={blocks}", flush=True)
    H = codes.rlc_H(n, n - m, seed=n + m)
    llr, _ = channel.awgn_llr(codes.generator_matrix(H), blocks, ebn0, seed=n * m)
    got = binding.orbg_decode(H, torch.from_numpy(llr).to(gpu_device), budget)
    _check(got, O.decode(H, llr, budget, THREADS), f"n={n} m={m}")


@pytest.mark.parametrize("budget", [1, 2, 63, 64, 65, 8191])
@pytest.mark.parametrize("blocks", [500, DIRECT + 2])
def test_dependent_columns_and_ties(gpu_device, blocks, budget):
    """Columns from a handful of values and zero columns, so that the eight least
    reliable ranks hold one to eight null combinations; magnitudes on a coarse
    grid in half of the blocks, so that ranks tie."""
    print(f"match dependent blocks={blocks} budget={budget}", flush=True)
    rng = np.random.default_rng(7)
    n, m = 100, 12
    pool = rng.integers(0, 2, size=(m, 9), dtype=np.uint8)
    pool[:, 0] = 0
    H = pool[:, rng.integers(0, 9, size=n)]
    H[:, :m] = np.eye(m, dtype=np.uint8)
    llr = (rng.standard_normal((blocks, n)) * 3).astype(np.float32)
    llr[::2] = np.round(llr[::2] * 2) / 2
    got = binding.orbg_decode(H, torch.from_numpy(llr).to(gpu_device), budget)
    _check(got, O.decode(H, llr, budget, THREADS), f"dependent {blocks} {budget}")


@pytest.mark.parametrize("budget", [64, 1000, 4096, 4097, 30000])
def test_batch_orders_that_repeat_or_leave_out_batches(gpu_device, budget):
    """A batch order is any 64 bytes (taken modulo 64): batches it leaves out are
    not tested, a repeated one counts again.  The expected results come from the
    oracle's pattern order, pattern by pattern."""
    print(f"match order budget={budget}", flush=True)
    rng = np.random.default_rng(budget)
    n, m, N = 90, 14, 150
    H = codes.rlc_H(n, n - m, seed=3)
    llr, _ = channel.awgn_llr(codes.generator_matrix(H), N, 3.0, seed=11)
    order = np.stack([rng.permutation(64) for _ in range(N)]).astype(np.uint8)
    order[::3, rng.integers(0, 64, 20)] = rng.integers(0, 64, 20)
    order[1::3] += 64 * rng.integers(0, 4, 64, dtype=np.uint8)
    got = binding.orbg_decode_ordered(H, torch.from_numpy(llr).to(gpu_device), budget,
                                      torch.from_numpy(order).to(gpu_device))
    pats = O.order_prefix_array(n, max(budget, 4096))
    cols = (H.astype(np.int64) << np.arange(m)[:, None]).sum(0)
    cw = (llr > 0).astype(np.uint8)
    q, ab = np.full(N, budget, dtype=np.uint64), np.ones(N, dtype=np.uint8)
    for b in range(N):
        perm = np.argsort(np.abs(llr[b]), kind="stable")
        h = np.concatenate([[0], cols[perm]])
        syn = np.bitwise_xor.reduce(cols * cw[b])
        member = np.bitwise_xor.reduce(h[pats], axis=1) == syn
        seq = np.concatenate([(order[b].astype(np.int64)[:, None] % 64 * 64 + np.arange(64)).reshape(-1),
                              np.arange(4096, len(pats))])[:budget]
        hit = np.nonzero(member[seq])[0]
        if hit.size:
            q[b], ab[b] = hit[0] + 1, 0
            ranks = pats[seq[hit[0]]]
            cw[b, perm[ranks[ranks > 0] - 1]] ^= 1
    _check(got, (cw, q, ab), f"order {budget}")


def test_mixed_codes_through_both_passes(gpu_device):
    """Five codes of three widths, one too short for the first pass, in one batch."""
    print("match mixed", flush=True)
    rng = np.random.default_rng(5)
    specs = [(11, 10), (64, 14), (100, 15), (127, 40), (250, 18)]
    Hs = [codes.rlc_H(n, n - m, seed=n) for n, m in specs]
    rows = []
    for H in Hs:
        llr, _ = channel.awgn_llr(codes.generator_matrix(H), 4000, 4.0, seed=H.shape[1])
        rows.append(llr)
    which = rng.permutation(np.repeat(np.arange(5), 4000)).astype(np.uint8)
    lens = np.array([n for n, _ in specs])[which]
    off = np.concatenate([[0], np.cumsum(lens)[:-1]]).astype(np.int64)
    flat = np.empty(int(lens.sum()), dtype=np.float32)
    at = [np.nonzero(which == i)[0] for i in range(5)]
    for i, (n, _) in enumerate(specs):
        flat[(off[at[i]][:, None] + np.arange(n)).reshape(-1)] = rows[i].reshape(-1)
    dev = gpu_device
    ids = [binding.orbg_code_register(H) for H in Hs]
    cw = torch.zeros(flat.size, dtype=torch.uint8, device=dev)
    q = torch.zeros(which.size, dtype=torch.int64, device=dev)
    ab = torch.zeros(which.size, dtype=torch.uint8, device=dev)
    binding.orbg_decode_mixed(ids, torch.from_numpy(which).to(dev), torch.from_numpy(off).to(dev),
                              torch.from_numpy(flat).to(dev), 2000, cw, q, ab)
    cw, q, ab = cw.cpu(), q.cpu(), ab.cpu()
    for i, (n, _) in enumerate(specs):
        idx = torch.from_numpy(off[at[i]])[:, None] + torch.arange(n)
        want = O.decode(Hs[i], rows[i], 2000, THREADS)
        _check((cw[idx], q[at[i]], ab[at[i]]), want, f"mixed n={n}")


@pytest.mark.parametrize("n,m,segments", [(9, 5, 1), (66, 30, 2), (200, 40, 4), (256, 20, 1), (300, 22, 3), (512, 20, 2)])
@pytest.mark.parametrize("curve", ["offset", "flat start", "steep start", "awgn"])
def test_mline_curves(gpu_device, n, m, segments, curve):
    """Magnitude curves that send the m-line match search through its parts: a
    large offset (every single rank before any pair, ranks past 254 among them),
    a nearly flat first segment (weights past the narrow tables, some past the
    wide ones), a steep one (offsets of the later segments below the first's
    end), and channel blocks; words at distance 1 to 4 from a codeword.  Every
    curve is noisy: on one that is linear to rounding the gaps of the fit are
    rounding errors, and the library evaluates its lines with one rounding less
    than the oracle."""
    print(f"mline curve {curve} n={n} m={m} segments={segments}", flush=True)
    rng = np.random.default_rng(n + len(curve))
    H = codes.rlc_H(n, n - m, seed=n)
    G = codes.generator_matrix(H)
    N = 64
    if curve == "awgn":
        llr, _ = channel.awgn_llr(G, N, 4.5, seed=n)
    else:
        r = np.arange(n, dtype=np.float64)
        mags = {"offset": 10.0 + 0.01 * r, "steep start": np.where(r < n // 8, 1.0 + r, 1.0 + n // 8 + 0.05 * (r - n // 8)),
                "flat start": np.where(r < max(3, n // 10), 0.5 + 1e-4 * r, 0.5 + 0.2 * (r - max(3, n // 10) + 1))}[curve]
        cw = channel.encode(G, rng.integers(0, 2, size=(N, G.shape[0]), dtype=np.uint8))
        llr = np.empty((N, n), dtype=np.float32)
        for b in range(N):
            perm = rng.permutation(n)
            rx = cw[b].copy()
            reach = n if b % 2 else max(4, n // 8)
            rx[perm[rng.choice(reach, size=1 + b % min(4, reach), replace=False)]] ^= 1
            llr[b, perm] = (mags * (1 + 1e-3 * (1 + b % 5) * rng.standard_normal(n))).astype(np.float32) * (2.0 * rx[perm] - 1)
    budget = min(40000, 2 ** n)
    got = binding.orbg_decode_mline(H, torch.from_numpy(llr).to(gpu_device), budget, segments)
    want = O.decode_mline(H, llr, budget, segments, threads=THREADS)
    _check(got[:3], want[:3], f"mline {curve} n={n}")
    assert (got[3].cpu().numpy() == want[3]).all()


def test_more_codewords_than_one_launch_addresses(gpu_device):
    """The first pass addresses codewords by 32-bit offsets, 2^30 bytes to a
    launch: a larger batch equals the same blocks decoded in two parts."""
    n, blocks, budget = 1024, (1 << 20) + 70, 200
    print(f"match slabs blocks={blocks}", flush=True)
    H = codes.rlc_H(n, n - 12, seed=5)
    g = torch.Generator(device=gpu_device).manual_seed(3)
    llr = torch.empty(blocks, n, device=gpu_device)
    for part in llr.split(1 << 17):
        part.normal_(-4.0, 2.0, generator=g)
    whole = binding.orbg_decode(H, llr, budget)
    half = blocks // 2 + 1
    for got, a, b in zip(whole, binding.orbg_decode(H, llr[:half], budget), binding.orbg_decode(H, llr[half:], budget)):
        assert torch.equal(got[:half], a) and torch.equal(got[half:], b)


@pytest.mark.parametrize("m", [8, 9])
def test_batch_orders_of_few_check_bits(gpu_device, m):
    """Both sides of the rule that sends an ordered decode to the match search."""
    print(f"match order m={m}", flush=True)
    H = codes.rlc_H(64, 64 - m, seed=m)
    llr, _ = channel.awgn_llr(codes.generator_matrix(H), 300, 3.0, seed=m)
    order = np.stack([np.random.default_rng(b).permutation(64) for b in range(300)]).astype(np.uint8)
    got = binding.orbg_decode_ordered(H, torch.from_numpy(llr).to(gpu_device), 6000, torch.from_numpy(order).to(gpu_device))
    _check(got, O.decode_ordered(H, llr, 6000, order, THREADS), f"order m={m}")
