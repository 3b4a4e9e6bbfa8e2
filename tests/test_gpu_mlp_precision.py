"""How far the surrogate's outputs are from 64 bits, in the mean over several
networks: bounds that the summation orders of the kernels have to keep."""
import numpy as np
import pytest

from oracle import mlp_oracle as M
from paper_2002_03120_amd import workloads as W

pytestmark = pytest.mark.gpu

NORM = np.array([0.2, 4.0, 2.75e-3, -4.6, 0.12, 1.15, 1.3e-3, 1.33], np.float32)


@pytest.fixture(scope="module")
def mlp():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_03120_amd import mlp
    mlp.lib()
    return mlp


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def test_error_of_the_inference(mlp):
    """Adding the parts of the activations chunk by chunk, six accumulations of
    the whole sum's size per layer, left 2.55e-7; four of the six are of smaller
    sums now, which leaves 2.0e-7 with the activations' own rounding."""
    off = []
    for seed in range(100, 116):
        p, x = W.mlp_init(seed), W.mlp_queries(4096, seed)
        y, ref = mlp.Mlp(p, NORM).predict(_dev(x)).cpu().numpy(), M.forward(p, x, NORM)
        off.append(np.linalg.norm(y - ref) / np.linalg.norm(ref))
    rms = float(np.sqrt(np.mean(np.square(off))))
    print(f"[case] 16 networks, 4096 rows: {rms:.3g}", flush=True)
    assert rms < 2.3e-7


def test_error_of_the_loss(mlp):
    """One rounding to 32 bits, below 2^-24 (2.5e-8 in the mean square with the
    mantissas spread evenly), and the residuals' own, which average out over
    the rows: 4e-8 at most."""
    off = []
    for seed in range(100, 164):
        p, x = W.mlp_init(seed), W.mlp_queries(256, seed)
        t = (2.5 * x[:, 0] + 4.0 * x[:, 0] ** 2).astype(np.float32)
        net = mlp.Mlp(p, NORM)
        net.train_step(_dev(x), _dev(t), update=False)
        ref, _ = M.loss_and_grad(p, x, t, NORM)
        off.append(net.read()[3] / ref - 1.0)
    rms = float(np.sqrt(np.mean(np.square(off))))
    print(f"[case] 64 networks, 256 rows: {rms:.3g}", flush=True)
    assert rms < 4e-8
