"""GPU checks of the network kernels where their paths change: the two inference
kernels and their ragged last tiles against each other, rows with NaN,
infinities, zeros and equal values, misaligned caller buffers; training at
batches around its row tiles and chunks against the fp64 reference."""
import numpy as np
import pytest
import torch

from oracle import mlp_ref as M
from paper_2202_13951_amd import binding, learned

pytestmark = pytest.mark.gpu
PERSIST = 24576                    # rows from which the weights stay in registers


def _net(dev, seed=3):
    return learned.Proposal(dev, w=torch.from_numpy(M.init(seed)))


def _rows(N, seed):
    rng = np.random.default_rng(seed)
    x = (rng.standard_normal((N, 128)) * 6).astype(np.float32)
    x[::7, ::5] = 0.0
    x[1::7] = np.round(x[1::7])
    x[2::11, 3] = np.inf
    x[3::13, 4] = np.nan
    x[3::13, 90] = np.frombuffer(np.uint32(0x7f812345).tobytes(), dtype=np.float32)[0]
    with np.errstate(invalid="ignore"):
        x[5::17] *= 1e-39
    return x


@pytest.mark.parametrize("N", [PERSIST - 1, PERSIST, PERSIST + 1, PERSIST + 127, 3 * 32768 + 5])
@pytest.mark.parametrize("shift", [0, 1])
def test_inference_kernels_agree(gpu_device, N, shift):
    """All N rows in one call against the same rows a few at a time (below the
    persistent kernel's size); features given (orbg_mlp_features) against
    features made; orders against orbg_mlp_order of the logits.  shift: llr and
    order start one element into their buffers."""
    print(f"infer N={N} shift={shift}", flush=True)
    p = _net(gpu_device)
    buf = torch.empty(N * 128 + 1, dtype=torch.float32, device=gpu_device)
    llr = buf[shift:shift + N * 128].view(N, 128)
    llr.copy_(torch.from_numpy(_rows(N, N)))
    lg = torch.empty((N, 64), dtype=torch.float32, device=gpu_device)
    ob = torch.empty(N * 64 + 1, dtype=torch.uint8, device=gpu_device)
    od = ob[shift:shift + N * 64].view(N, 64)
    binding.orbg_mlp_infer(p.w, p.wb, llr=llr, logits=lg, order=od)
    part, x = torch.empty_like(lg), learned.features(llr.clone())
    for s in range(0, N, 9000):
        e = min(N, s + 9000)
        binding.orbg_mlp_infer(p.w, p.wb, llr=llr[s:e].contiguous(), logits=part[s:e])
    fx, fo = torch.empty_like(lg), torch.empty((N, 64), dtype=torch.uint8, device=gpu_device)
    binding.orbg_mlp_infer(p.w, p.wb, x=x, logits=fx, order=fo)
    want = torch.empty((N, 64), dtype=torch.uint8, device=gpu_device)
    binding.orbg_mlp_order(lg, want)
    torch.cuda.synchronize()
    same = lambda a, b: torch.equal(a.view(torch.int32), b.view(torch.int32))   # noqa: E731  (NaN rows too)
    assert same(lg, part) and same(lg, fx)
    assert torch.equal(od, want) and torch.equal(fo, want)


def test_orders_of_close_and_special_logits(gpu_device):
    """Logits that share their leading bits, equal ones, zeros of both signs,
    infinities and NaN: a network whose last layer has no weights gives its
    biases as logits."""
    print("orders of close logits", flush=True)
    rng = np.random.default_rng(2)
    p = _net(gpu_device)
    for k in range(12):
        b = rng.standard_normal(64).astype(np.float32)
        if k % 3 == 0:
            b = (1.0 + np.float32(2.0 ** -23) * rng.integers(0, 40, 64)).astype(np.float32)
        if k % 3 == 1:
            b[rng.integers(0, 64, 20)] = rng.choice(np.array([0.0, -0.0, np.inf, -np.inf, np.nan, 1.0], np.float32), 20)
        w = p.w.clone()
        w[-64 * 256 - 64:-64] = 0.0
        w[-64:] = torch.from_numpy(b).to(gpu_device)
        q = learned.Proposal(gpu_device, w=w)
        od = torch.empty((3, 64), dtype=torch.uint8, device=gpu_device)
        binding.orbg_mlp_infer(q.w, q.wb, llr=torch.ones((3, 128), device=gpu_device), order=od, pin0=bool(k & 1))
        want = M.order(b[None, :])[0]
        if k & 1:
            want = np.concatenate([[0], want[want != 0]])
        assert (od.cpu().numpy() == want).all(), k


@pytest.mark.parametrize("N", [1, 31, 32, 33, 511, 513, 16385])
def test_training_batches(gpu_device, N):
    """Gradients of every layer and the loss around the row tiles (32) and the
    chunks of the weight gradients (512): the FP64 reference with the same BF16
    roundings, within the tolerance of BF16 values near a rounding edge."""
    print(f"train N={N}", flush=True)
    p = _net(gpu_device, 5)
    rng = np.random.default_rng(N)
    llr = (rng.standard_normal((N, 128)) * 6).astype(np.float32)
    labels = rng.integers(0, 64, N).astype(np.int32)
    x = learned.features(torch.from_numpy(llr).to(gpu_device))
    p.grads.fill_(float("nan"))
    ws = p.workspace(N)
    ws.fill_(0xff)                  # every value the kernels read has to be written first
    binding.orbg_mlp_backward(p.w, p.wb, p.wt, x, torch.from_numpy(labels).to(gpu_device), p.grads, p.loss, ws)
    torch.cuda.synchronize()
    loss, ref = M.backward(p.w.cpu().numpy(), x.view(torch.bfloat16).float().cpu().numpy(), labels)
    assert abs(float(p.loss.item()) - loss) <= 1e-3 * abs(loss)
    G, R = M.unflatten(p.grads.cpu().numpy().astype(np.float64)), M.unflatten(ref)
    for name, _ in M.SHAPES:
        a, b = G[name].reshape(-1), R[name].reshape(-1)
        assert np.linalg.norm(a - b) <= 3e-2 * np.linalg.norm(b), name
