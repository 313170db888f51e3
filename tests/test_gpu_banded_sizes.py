"""The time-banded epilogue at its edges (one and several rounds of 16 and 64
(block, mode) pairs, the largest count of both, basis sizes that are no multiple
of its unrolled reads) against the oracle's online stage on the library's own
artefacts."""
import numpy as np
import pytest

from oracle import likelihood as lk
from oracle import startup as su
from paper_2508_04172_amd import rbfl
from paper_2508_04172_amd import workloads as wl

from test_gpu_banded import run

pytestmark = pytest.mark.gpu

SITES = wl.SITES_HLV + wl.SITE_GEOCENTRE


@pytest.mark.parametrize("n_det, n_modes, n_bands, q", [(1, 1, 2, 13), (1, 5, 3, 8), (2, 4, 2, 1), (3, 5, 4, 17),
                                                       (3, 2, 11, 9), (4, 5, 16, 7)])
def test_matches_oracle(n_det, n_modes, n_bands, q):
    cfg = wl.SMALL_BANDED.with_(name="banded_sizes", sites=SITES[:n_det], modes=wl.ALL_MODES[:n_modes],
                                n_bands=n_bands, n_nodes=60, q=q)
    inj = wl.injection_extrinsics(cfg)
    h = rbfl.Handle.from_config(cfg, wl.white_noise(cfg), inj)
    art = su.artefacts_from_exports(cfg, inj, **h.exports())
    n = 131
    idx, jit = wl.node_jitter(n, cfg.n_nodes, seed=q)
    qd = wl.queries(cfg, n=n, seed=q).near_nodes(h.nodes(), idx, jit)
    P = np.ascontiguousarray(rbfl.params_soa(h, qd, cfg.t_trig))
    P[9, 5] = cfg.t_trig + 10.0                       # outside the window
    P[6, 7] = np.nan
    got = run(h, P)
    want = lk.meshfree_lnl(art, P[0:4].T.copy(), P[4:9].T.copy(), P[9].copy(), P[10].copy())
    assert np.isnan(got[7]) and got[5] == -np.inf
    keep = np.arange(n) != 7
    fin = np.isfinite(want) & keep
    assert fin.sum() >= n // 2 and np.array_equal(fin[keep], np.isfinite(got[keep]))
    # the bar of the other evaluation-parity tests on the same artefacts
    assert np.abs(got[fin] - want[fin]).max() <= 1e-3 * max(1.0, np.abs(want[fin]).max() * 1e-6)
