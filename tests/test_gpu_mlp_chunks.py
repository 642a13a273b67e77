"""The training kernel's chunking: batches at the edges of its 32-row chunks and
of its workgroups' chunk counts, against the CPU oracle."""
import numpy as np
import pytest

import oracle
from test_gpu_mlp import _data, _term_magnitudes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# one row; a chunk less, exactly and more than one row; 64 chunks (one per
# workgroup) plus a row; 2 and then 4 chunks per workgroup with a ragged last one
@pytest.mark.parametrize("n", [1, 31, 33, 2049, 4100, 9001])
def test_gradient_and_step_at_chunk_edges(n):
    """Gradient within 1e-2 of the oracle's plus 2^-7 of each entry's term
    magnitude (one-ulp bfloat16 differences of both operands), loss within
    1e-3; a training step moves the parameters by the oracle's Adam step on
    that gradient; inputs at an address that is only 4-byte aligned give the
    same bits."""
    import torch
    import paper_2609_30459_amd as vf
    P = oracle.mlp_init(21)
    X, T = _data(n, 300 + n)
    L_o, G_o, _ = oracle.mlp_loss_grad(P, X, T)
    A = _term_magnitudes(P, X, T)
    with vf.Mlp(n) as net:
        net.set_params(P)
        dx, dt = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
        g = torch.zeros(vf.MLP_NPARAM, dtype=torch.float32, device="cuda")
        L_g = net.gradient(dx, dt, g)
        G_g = g.cpu().numpy()
        assert abs(L_g - L_o) <= 1e-3 * abs(L_o)
        err = np.abs(G_g.astype(np.float64) - G_o)
        bad = np.nonzero(err > 1e-2 * np.abs(G_o) + 2.0 ** -7 * A)[0]
        assert not len(bad), (len(bad), G_g[bad[:5]].tolist(), G_o[bad[:5]].tolist(), A[bad[:5]].tolist())
        shifted = torch.zeros(n * 32 + 1, device="cuda")
        shifted[1:] = dx.reshape(-1)
        g2 = torch.zeros_like(g)
        assert net.gradient(shifted[1:].view(n, 32), dt, g2) == L_g
        assert torch.equal(g, g2)
        want, m, v = P.copy(), np.zeros_like(P), np.zeros_like(P)
        oracle.adam(want, G_g, m, v, 1, lr=1e-3)
        assert net.train_step(dx, dt, lr=1e-3) == L_g
        got = net.get_params()
    move = want.astype(np.float64) - P
    tol = 1e-2 * np.abs(move) + 2.0 ** -22 * np.abs(P)
    assert (np.abs(got.astype(np.float64) - want) <= tol).all()


# more chunks than workgroups (512) with a ragged last one; exactly two rounds; one row
@pytest.mark.parametrize("n", [1, 33, 16385, 32768])
def test_forward_at_chunk_edges(n):
    """Outputs within 2e-2 of the mean magnitude of the oracle's (bfloat16
    flips), the median within 1e-3 of it, and nothing written past row n."""
    import torch
    import paper_2609_30459_amd as vf
    P = oracle.mlp_init(23)
    P[-3:] = [0.05, -0.02, 0.1]
    X, _ = _data(n, 500 + n)
    want, _, _ = oracle.mlp_forward(P, X)
    with vf.Mlp(16) as net:
        net.set_params(P)
        y = torch.full((n + 8, 3), 7.0, device="cuda")
        net.forward(torch.from_numpy(X).cuda(), y)
        got = y.cpu().numpy()
    assert (got[n:] == 7.0).all()
    scale = np.abs(want).mean() + 1e-3
    err = np.abs(got[:n] - want)
    assert err.max() <= 2e-2 * scale and np.median(err) <= 1e-3 * scale, (err.max(), scale)
