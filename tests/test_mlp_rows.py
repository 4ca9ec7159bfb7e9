"""The gradient sums of the network kernels, on samples where every tile of 16
counts: one row of each tile (a place that moves from tile to tile) and every
row of the ragged last tile have targets a hundred times the others', so that
one of them left out, or taken twice, moves every layer's block of the gradient
by more than 4e-2 of the block's largest entry (checked on the reference).

Tolerance 1e-2 of each block's largest entry: kernel and reference round at the
same points, so they part where an FP32 sum lies on the other side of a bfloat16
boundary than the FP64 one, an ulp (2^-8 relative) in one row's share of a block:
4e-3 where a block is one row.  Offsets of 2^-21 in the reference's biases,
which stand for the FP32 sums, move no block by more than 1.4e-3."""
import numpy as np
import pytest

from oracle import surrogate as S

SIZES = [1, 15, 17, 256, 257, 512, 529, 771]
TOL, SEEN = 1e-2, 4e-2


def _case(n):
    from paper_2403_05443_amd import workloads
    g = np.random.default_rng(7000 + n)
    p = workloads.xavier_params(workloads.SplitMix64(900 + n)).astype(np.float32)
    p += g.uniform(-0.1, 0.1, p.shape).astype(np.float32)
    X = g.uniform(-1, 1, (n, 8)).astype(np.float32)
    Y = g.uniform(-1, 1, (n, 6)).astype(np.float32)
    t = np.arange((n + 15) // 16)
    heavy = np.unique(np.concatenate([(16 * t + (5 * t) % 16)[:-1], np.arange(16 * t[-1], n)]))
    Y[heavy] *= 100
    return p, X, Y, heavy


def _reference(p, X, Y):
    return S.loss_grad(p.astype(np.float64), X.astype(np.float64), Y.astype(np.float64), bf=True)


def _apart(g, ref):
    """Largest difference of each layer's block, in units of the block's largest entry."""
    a, b = S.unpack(np.asarray(g, dtype=np.float64)), S.unpack(ref)
    return {k: np.abs(a[k] - b[k]).max() / np.abs(b[k]).max() for k in b}


@pytest.mark.parametrize("n", SIZES[1:])
def test_each_heavy_row_shows_in_every_block(n):
    p, X, Y, heavy = _case(n)
    _, ref = _reference(p, X, Y)
    for r in heavy:
        keep = np.arange(n) != r
        _, g = _reference(p, X[keep], Y[keep])
        assert min(_apart(g * (n - 1) / n, ref).values()) > SEEN, r


@pytest.mark.gpu
@pytest.mark.parametrize("n", SIZES)
def test_every_row_once(n):
    import torch
    from paper_2403_05443_amd import lbell
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    p, X, Y, _ = _case(n)
    L, g = lbell.Surrogate(max_samples=n, params=p).grad(X, Y)
    Lr, gr = _reference(p, X, Y)
    assert abs(L - Lr) < 1e-3 * Lr
    apart = _apart(g, gr)
    print(n, {k: f"{v:.1e}" for k, v in apart.items()})
    assert max(apart.values()) < TOL, apart
