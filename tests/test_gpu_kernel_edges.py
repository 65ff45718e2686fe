"""Kernels at the sizes where their tilings can go wrong (edges, remainders, smallest and largest
of a range), against the oracle or plain FP64 definitions."""

import numpy as np
import pytest

from paper_2406_14542_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def rel(a, b):
    return float(np.linalg.norm(np.ravel(a - b)) / np.linalg.norm(np.ravel(b)))


@pytest.fixture(scope="module")
def P():
    import paper_2406_14542_amd as P
    P.lib()
    return P


SIZES = [12, 128, 128, 128, 1]


@pytest.mark.parametrize("n", [15, 16, 17, 32, 33, 16383, 16385, 16449, 32832])
def test_mlp_tiles(P, oracle_mod, n):
    """Tiles of 64 points (blocks of 16, halves of 32), up to 256 blocks that stride over the
    tiles.  FP32 sums of up to 128 terms per layer and, for the gradient, 64-point tile sums:
    rounding 2^-24 sqrt(128) per layer, four layers, is below 3e-6; 1e-5 and 2e-5 leave room for
    the functions' own ulp."""
    print(f"[mlp n={n}]", flush=True)
    rng = np.random.default_rng(n)
    flat32 = oracle_mod.mlp_pack(oracle_mod.mlp_init(SIZES, seed=3)).astype(np.float32)
    p64 = oracle_mod.mlp_unpack(flat32.astype(np.float64), SIZES)
    X = rng.standard_normal((n, 12)).astype(np.float32)
    gy = (0.5 + rng.uniform(size=n)).astype(np.float32)
    y = P.mlp_forward(dev(flat32), dev(X), 0.37).cpu().numpy()
    yw, cache = oracle_mod.mlp_forward(p64, X.astype(np.float64), 0.37)
    assert y.shape == (n,) and rel(y, yw) <= 1e-5, rel(y, yw)
    g = P.mlp_backward(dev(flat32), dev(X), dev(gy), 0.37).cpu().numpy()
    gw = oracle_mod.mlp_pack(oracle_mod.mlp_backward(p64, cache, gy.astype(np.float64), 0.37))
    assert rel(g, gw) <= 2e-5, rel(g, gw)
    # every point counts once: the output bias's gradient is the sum of the points' terms alone
    assert abs(g[-1] - gw[-1]) <= 2e-5 * abs(gw[-1])
