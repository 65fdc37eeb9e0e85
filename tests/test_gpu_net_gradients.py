"""The warm-start network's FP32 forward and gradients on MFMA against the FP64 oracle, at the
edges of the kernels' tiles: 64 output channels, 16 input channels, 32 and 128 positions, a
position count past a multiple of 4, every tap count, more chunks than partial sums.

Tolerances are those of the network's other tests: FP32 sums of at most 15 x 130 terms a layer give
outputs to 1e-5 relative; the gradients pass through the forward's and the backward's layers and
sum up to 5 x 1300 positions: 1e-4.
"""
import numpy as np
import pytest

from oracle import warmstart_ref as wr
from parity import rel

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2503_00253_amd import infoesrf as ie  # noqa: E402

D = 4


def flat(params):
    return np.concatenate([np.concatenate([W.ravel(), b.ravel()]) for W, b in params])


@pytest.mark.parametrize("H,K,B,m", [(1, 1, 1, 1), (4, 3, 2, 3), (16, 5, 3, 32), (17, 7, 2, 33), (63, 9, 2, 127),
                                     (64, 9, 1, 128), (65, 11, 2, 129), (72, 13, 1, 130), (130, 15, 1, 70),
                                     (64, 9, 5, 1300), (8, 15, 80, 9)])
def test_forward_and_gradients_at_tile_edges(H, K, B, m):
    rng = np.random.default_rng(H * 1000 + K * 100 + m)
    params = wr.init_params(channels=(1, H, H, H, D), K=K, seed=K)
    params = [(W.astype(np.float32).astype(np.float64),
               (0.05 * rng.standard_normal(b.shape)).astype(np.float32).astype(np.float64)) for W, b in params]
    net = ie.Net.create(H, K, 1)
    net.set_params(flat(params).astype(np.float32))
    Q = 3
    X = rng.standard_normal((B, m)).astype(np.float32)
    cq = np.array([0.9, 0.4, 0.05], dtype=np.float32)
    T = rng.standard_normal((B, Q, m)).astype(np.float32)
    Xd, cd, Td = (torch.from_numpy(a).cuda() for a in (X, cq, T))
    Y, _ = wr.forward(params, X.astype(np.float64)[:, None, :])
    assert rel(net.forward(Xd).cpu().numpy(), Y) < 1e-5
    got, loss = net.gradients(Xd, cd, Td)
    c = cq.astype(np.float64)
    phi = np.stack([c ** (d + 1) for d in range(D)], axis=1)
    Y, cache = wr.forward(params, X.astype(np.float64)[:, None, :])
    want_loss, gy = wr.loss_rel_l2(wr.head(Y, phi), T.astype(np.float64))
    grads = wr.backward(params, cache, wr.head_grad(gy, phi))
    assert abs(float(loss) - want_loss) < 1e-5 * max(1.0, want_loss)
    assert rel(got.cpu().numpy(), flat(grads)) < 1e-4


@pytest.mark.parametrize("H,K,B,m", [(16, 9, 9, 1021), (17, 1, 33, 2049), (24, 9, 40, 500), (31, 5, 40, 433),
                                     (40, 7, 33, 511), (40, 15, 40, 433), (64, 9, 20, 900), (130, 11, 20, 333)])
def test_forward_and_gradients_where_layers_leave_the_matrix_cores(H, K, B, m):
    """Batches past the blocks up to which narrow layers run on the matrix cores: hidden layers and the
    last one with FP32 FMAs, 16 or 4 output channels a block, 64 positions, the last chunk of input
    channels not full."""
    test_forward_and_gradients_at_tile_edges(H, K, B, m)
