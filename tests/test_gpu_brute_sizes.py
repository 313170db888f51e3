"""The exact ln L at every detector count and on both workgroup sizes, against
the oracle's brute force."""
import types

import numpy as np
import pytest

from oracle import startup as su
from paper_2508_04172_amd import rbfl
from paper_2508_04172_amd import workloads as wl

from test_gpu_brute import gpu_brute, oracle_brute

pytestmark = pytest.mark.gpu

SITES = wl.SITES_HLV + wl.SITE_GEOCENTRE


# one workgroup of 16 waves per proposal up to 512 proposals, 4 waves above;
# 1, 3 and 5 modes; a segment whose bins are no multiple of either
@pytest.mark.parametrize("n", [1, 512, 513])
@pytest.mark.parametrize("n_det, n_modes", [(1, 1), (2, 3), (3, 5), (4, 2)])
def test_matches_oracle(n_det, n_modes, n):
    cfg = wl.SMALL_MULTI.with_(name="brute_sizes", seg_len=4.0, f_low=25.0, sites=SITES[:n_det],
                               modes=wl.ALL_MODES[:n_modes], n_nodes=40, q=8)
    white, inj = wl.white_noise(cfg), wl.injection_extrinsics(cfg)
    h = rbfl.Handle.from_config(cfg, white, inj)
    idx, jit = wl.node_jitter(n, cfg.n_nodes, seed=n)
    p = rbfl.params_soa(h, wl.queries(cfg, n=n, seed=n).near_nodes(h.nodes(), idx, jit), cfg.t_trig)
    got = gpu_brute(h, p)
    pick = np.unique(np.linspace(0, n - 1, 12).astype(int))
    want = oracle_brute(types.SimpleNamespace(ev=su.make_event(cfg, white, inj)), h, p[:, pick], cfg)
    fin = np.isfinite(want)
    assert np.array_equal(fin, np.isfinite(got[pick]))
    # both sum the same band in 64 bits: rounding only, as in the other tests of this path
    assert np.all(np.abs(got[pick][fin] - want[fin]) <= 1e-9 * np.maximum(1.0, np.abs(want[fin])))
