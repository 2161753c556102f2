"""GPU parity with the CPU oracle on paths that the other tests' sizes do not reach:
the first pass (batches above 24576 blocks) of mixed codes, of special values and
into views of larger buffers, its longest groups; the search by steps and its heavy
pass in a mixed launch, which one code of n <= 8 sends all codes to; both inference
kernels against the fp64 network."""
import os

import numpy as np
import pytest
import torch

from oracle import mlp_ref as M
from oracle import oracle as O
from paper_2202_13951_amd import binding, learned
from synth import channel, codes

pytestmark = pytest.mark.gpu
THREADS = min(16, os.cpu_count() or 1)
DIRECT = 24576                       # largest batch decoded by one launch
PERSIST = 24576                      # rows from which the network's weights stay in registers


def _same(got, want, tag):
    cw, q, ab = got
    bad = np.nonzero((cw != want[0]).any(axis=1) | (q.astype(np.uint64) != want[1]) | (ab != want[2]))[0]
    assert bad.size == 0, f"{tag}: {bad.size} differ, first {bad[:8].tolist()}: gpu {q[bad[:4]]} oracle {want[1][bad[:4]]}"


def _mixed_case(specs, blocks, ebn0, seed):
    """Shuffled blocks of several codes in one buffer: matrices, block codes, row
    offsets, LLRs."""
    rng = np.random.default_rng(seed)
    Hs = [codes.rlc_H(n, n - m, seed=n) for n, m in specs]
    which = rng.permutation(np.arange(blocks) % len(specs)).astype(np.uint8)
    lens = np.array([n for n, _ in specs])[which]
    off = np.concatenate([[0], np.cumsum(lens)[:-1]]).astype(np.int64)
    flat = np.empty(int(lens.sum()), dtype=np.float32)
    for i, (n, _) in enumerate(specs):
        at = np.nonzero(which == i)[0]
        llr, _ = channel.awgn_llr(codes.generator_matrix(Hs[i]), at.size, ebn0, seed=seed + n)
        flat[off[at][:, None] + np.arange(n)] = llr
    return Hs, which, off, flat


def _check_mixed(dev, Hs, which, off, flat, budget, tag, outside=None, params=None):
    """Decodes the case and compares every block with the oracle.  outside: blocks
    whose row is moved out of the buffer, {block: offset}."""
    ids = [binding.orbg_code_register(H) for H in Hs]
    moved = off.copy()
    for b, o in (outside or {}).items():
        moved[b] = o
    cw = torch.full((flat.size,), 7, dtype=torch.uint8, device=dev)
    q = torch.full((which.size,), -1, dtype=torch.int64, device=dev)
    ab = torch.full((which.size,), 9, dtype=torch.uint8, device=dev)
    binding.orbg_decode_mixed(ids, torch.from_numpy(which).to(dev), torch.from_numpy(moved).to(dev),
                              torch.from_numpy(flat).to(dev), budget, cw, q, ab, params=params)
    cw, q, ab = cw.cpu().numpy(), q.cpu().numpy(), ab.cpu().numpy()
    code = np.where(which < len(Hs), which, 0)           # out-of-range indices decode with code 0
    inside = np.ones(which.size, dtype=bool)
    for b in outside or {}:
        inside[b] = False
        n = Hs[code[b]].shape[1]
        assert q[b] == 1 and ab[b] == 0 and (cw[off[b]:off[b] + n] == 7).all(), (tag, b)
    for i, H in enumerate(Hs):
        at = np.nonzero((code == i) & inside)[0]
        rows = off[at][:, None] + np.arange(H.shape[1])
        _same((cw[rows], q[at], ab[at]), O.decode(H, np.ascontiguousarray(flat[rows]), budget, THREADS),
              f"{tag} n={H.shape[1]}")
    for i in ids:
        binding.orbg_code_release(i)
    return q


def test_mixed_first_pass(gpu_device):
    """Five codes of three widths above the one-launch batch size: n = 11 (left to the
    search), a 64-bit syndrome, rows outside the buffers and indices past the codes."""
    print("mixed first pass", flush=True)
    specs = [(11, 10), (64, 14), (100, 15), (127, 40), (250, 18)]
    blocks = 5 * (DIRECT // 5 + 900)
    assert blocks > DIRECT
    Hs, which, off, flat = _mixed_case(specs, blocks, 4.0, 5)
    rng = np.random.default_rng(6)
    some = rng.choice(np.nonzero(which != 0)[0], 60, replace=False)
    where = [-1, -(1 << 40), flat.size - 8, flat.size, 1 << 40]
    outside = {int(b): where[i % 5] for i, b in enumerate(some[:40])}
    first = np.nonzero(which == 0)[0]
    which[first[::7]] = 5 + (np.arange(first[::7].size) % 250)
    _check_mixed(gpu_device, Hs, which, off, flat, 2000, "mixed", outside)


@pytest.mark.parametrize("blocks", [9000, DIRECT + 3500])
def test_mixed_with_a_short_code_goes_by_steps(gpu_device, blocks):
    """One code of n = 7 among wide ones: the light and the heavy pass decode them all,
    in every launch shape."""
    print(f"mixed by steps blocks={blocks}", flush=True)
    specs = [(64, 12), (7, 3), (128, 16), (200, 17)]
    Hs, which, off, flat = _mixed_case(specs, blocks, 4.0, 8)
    shapes = [None, dict(split_steps=1, heavy_waves=4), dict(split_steps=3, heavy_waves=16, heavy_workgroups_per_cu=1),
              dict(split_steps=0), dict(workgroups_per_cu=2, chunk=5, split_steps=8), dict(one_block_per_workgroup=1)]
    for shape in shapes if blocks < DIRECT else shapes[:3]:
        q = _check_mixed(gpu_device, Hs, which, off, flat, 20000, f"by steps {shape}",
                         params=binding.LaunchParams(**shape) if shape else None)
        assert (q > 64 * 64).any()                       # the heavy pass took part, where there is one


@pytest.mark.parametrize("n,m,blocks", [(48, 10, 256 * 32 * 16 + 77), (64, 12, 256 * 32 * 16 + 1), (127, 14, 256 * 32 * 8 + 5),
                                        (300, 20, DIRECT + 901)])
def test_first_pass_special_rows_and_views(gpu_device, n, m, blocks):
    """Runs of rows of zeros, infinities, NaN, equal magnitudes and very large and small
    scales among ordinary ones (each wave's threshold has to come back from them); the
    outputs are views with sentinel rows on both sides.  The sizes take the pass's
    longest groups at one and two keys per lane."""
    print(f"first pass n={n} blocks={blocks}", flush=True)
    rng = np.random.default_rng(n)
    H = codes.rlc_H(n, n - m, seed=n)
    llr, _ = channel.awgn_llr(codes.generator_matrix(H), blocks, 4.0, seed=n)
    special = [lambda x: x * 0, lambda x: -0.0 * np.abs(x), lambda x: np.sign(x) * np.float32(np.inf),
               lambda x: np.where(rng.random(x.shape) < 0.2, np.float32(np.nan), x), lambda x: np.sign(x) * 2,
               lambda x: x * np.float32(1e-42), lambda x: x * np.float32(1e30), lambda x: np.round(x),
               lambda x: np.where(rng.random(x.shape) < 0.3, np.float32(-np.inf), x)]
    with np.errstate(invalid="ignore", over="ignore"):
        for r in range(60):
            s = int(rng.integers(0, blocks - 80))
            e = s + int(rng.integers(1, 80))
            llr[s:e] = special[r % len(special)](llr[s:e])
    llr = llr.astype(np.float32)
    big = torch.full((blocks + 2, n), -40.0, dtype=torch.float32, device=gpu_device)
    big[1:-1] = torch.from_numpy(llr).to(gpu_device)
    cw = torch.full((blocks + 2, n), 7, dtype=torch.uint8, device=gpu_device)
    q = torch.full((blocks + 2,), -1, dtype=torch.int64, device=gpu_device)
    ab = torch.full((blocks + 2,), 9, dtype=torch.uint8, device=gpu_device)
    binding.orbg_decode(H, big[1:-1], 400, out=(cw[1:-1], q[1:-1], ab[1:-1]))
    cw, q, ab = cw.cpu().numpy(), q.cpu().numpy(), ab.cpu().numpy()
    for r in (0, -1):
        assert (cw[r] == 7).all() and q[r] == -1 and ab[r] == 9
    _same((cw[1:-1], q[1:-1], ab[1:-1]), O.decode(H, llr, 400, THREADS), f"first pass n={n}")


@pytest.mark.parametrize("N", [33, PERSIST - 1, PERSIST + 37])
def test_inference_kernels_match_the_reference(gpu_device, N):
    """Both inference kernels and orbg_mlp_forward (which is one of them) against the
    fp64 network: each row's logits to 1e-2 of its largest (BF16 activations that fall
    on the other side of a rounding boundary)."""
    print(f"inference against fp64 N={N}", flush=True)
    rng = np.random.default_rng(N)
    d = M.unflatten(M.init(4).astype(np.float64))
    for b in ("b1", "b2", "b3"):
        d[b][:] = rng.standard_normal(d[b].shape) * 0.1
    w = M.flatten(d).astype(np.float32)
    p = learned.Proposal(gpu_device, w=torch.from_numpy(w))
    llr = (rng.standard_normal((N, 128)) * 6).astype(np.float32)
    ref, _ = M.forward(w, M.features(llr))
    x = torch.from_numpy(llr).to(gpu_device)
    lg = torch.empty((N, 64), dtype=torch.float32, device=gpu_device)
    binding.orbg_mlp_infer(p.w, p.wb, llr=x, logits=lg)
    for got in (lg, p.logits(learned.features(x))):
        err = np.abs(got.cpu().numpy() - ref).max(axis=1) / np.abs(ref).max(axis=1)
        assert (err <= 1e-2).all(), float(err.max())


@pytest.mark.parametrize("which", ["two passes", "few check bits", "small m-line"])
def test_graph_replay_of_the_search_kernels(gpu_device, which):
    """Captured decodes whose kernels the other replay tests do not hold: the first pass
    and the match search behind it, the kernel for few check bits, the one-launch
    m-line decode.  Every replay, with eager work in between, equals the eager result."""
    print(f"graph replay {which}", flush=True)
    n, m, blocks = {"two passes": (100, 14, DIRECT + 3000), "few check bits": (90, 2, 900), "small m-line": (150, 16, 500)}[which]
    H = codes.rlc_H(n, n - m, seed=n)
    llr, _ = channel.awgn_llr(codes.generator_matrix(H), blocks, 4.0, seed=n)
    x = torch.from_numpy(llr).to(gpu_device)
    out = (torch.zeros((blocks, n), dtype=torch.uint8, device=gpu_device),
           torch.zeros(blocks, dtype=torch.int64, device=gpu_device), torch.zeros(blocks, dtype=torch.uint8, device=gpu_device))

    def call(rows, dst, stream=None):
        if which == "small m-line":
            binding.orbg_decode_mline(H, rows, 3000, 3, segments_out=False, out=dst, stream=stream)
        else:
            binding.orbg_decode(H, rows, 3000, out=dst, stream=stream)

    call(x, out)
    eager = [t.clone() for t in out]
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        call(x, out, s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        call(x, out, s)
    other = [torch.empty_like(t) for t in out]
    for rep in range(3):
        for t, v in zip(out, (7, -1, 9)):
            t.fill_(v)
        call(x.flip(0).contiguous(), other)
        g.replay()
        torch.cuda.synchronize()
        for t, want, swapped in zip(out, eager, other):
            assert torch.equal(t, want) and torch.equal(swapped.flip(0), want), rep
