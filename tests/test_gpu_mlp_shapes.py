"""The surrogate network's products at shapes with tile remainders, on both
tile sizes, against the oracle: forward, loss and every gradient."""
import numpy as np
import pytest

from oracle import mlp as omlp
from paper_2508_04172_amd import rbfl
from paper_2508_04172_amd import workloads as wl

pytestmark = pytest.mark.gpu


# (inputs, hidden, outputs, samples): below one tile, one past a tile of 32 and of
# 64, rows that are not 16-byte aligned, more inputs than the first layer's own
# kernels take, enough tiles for 64 x 64 and for the 128 x 128 forward layers
@pytest.mark.parametrize("n_in, hidden, n_out, B", [
    (4, 8, 1, 1), (1, 9, 2, 3), (4, 33, 37, 31), (4, 32, 64, 64), (4, 65, 129, 97), (3, 100, 131, 257),
    (7, 64, 41, 130), (8, 48, 70, 100), (20, 36, 66, 95), (4, 256, 1275, 1024), (4, 100, 1275, 2049),
    (4, 128, 600, 4100)])
def test_products_match_oracle(n_in, hidden, n_out, B):
    import torch
    z = wl.mlp_normals(rbfl.mlp_param_count(n_in, hidden, n_out))
    rng = np.random.default_rng(B)
    X = rng.uniform(-1, 1, (B, n_in)).astype(np.float32)
    T = rng.standard_normal((B, n_out)).astype(np.float32)
    net = rbfl.Mlp(n_in, hidden, n_out, z)
    xg, tg = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
    y = torch.empty(B, n_out, dtype=torch.float32, device="cuda")
    net.forward(xg.data_ptr(), B, y.data_ptr())
    loss = net.loss_grad(xg.data_ptr(), tg.data_ptr(), B)
    g = net.get(1)
    vec = net.get(0).astype(np.float64)               # the FP32 parameters in use
    Yo, _ = omlp.forward(vec, X.astype(np.float64), n_in, hidden, n_out)
    Lo, go = omlp.loss_and_grad(vec, X.astype(np.float64), T.astype(np.float64), n_in, hidden, n_out)
    # FP32 sums of at most 4100 terms in groups of 16 or 32: 2^-24 sqrt(4100) = 4e-6 of
    # the largest value, plus the hardware exponential's few 1e-7
    assert np.abs(y.cpu().numpy() - Yo).max() <= 1e-5 * max(1.0, np.abs(Yo).max())
    assert loss == pytest.approx(Lo, rel=1e-5)
    assert np.abs(g - go).max() <= 1e-5 * np.abs(go).max()
    net.close()
