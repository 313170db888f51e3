"""The time-banded epilogue alone: ln L from the library's own interpolated
outputs against the oracle's combination of the same outputs, to the rounding of
the sums, at batch sizes around its change of NaN counting (4096 proposals)."""
import numpy as np
import pytest

from oracle import likelihood as lk
from oracle import startup as su
from paper_2508_04172_amd import rbfl
from paper_2508_04172_amd import workloads as wl

from test_gpu_banded import run

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -52


def rounding_bound(cfg, art, Y, d_l):
    """Per proposal, what two FP64 evaluations of ln L from outputs Y can differ
    by: EPS times the sum of the absolute terms, S, for each of the roundings a
    term goes through (below 200: q <= 17 products and as many additions, 10
    spline taps in 4 powers, harmonics of up to 8 factors, antenna factors), and
    the arrival-time position's own rounding, EPS (t_trig + 2 s) fs samples,
    through the spline's slope.  |A| <= 1: |F+ + i Fx| <= 1, |Y_lm| <= 0.85."""
    n_v, nm = cfg.n_det * cfg.n_bands, len(cfg.modes)
    _, coef_off, sig_off = su.output_layout(n_v, nm, art.q)
    f = np.linspace(0.0, 1.0, 101)
    tab = lk.spline_table()
    weights = np.abs(lk.spline_weights(f, tab)).sum(1).max()
    slope = np.abs(tab[None, :, 1] + f[:, None] * (2 * tab[None, :, 2] + 3 * f[:, None] * tab[None, :, 3])).sum(1).max()
    r = art.d_ref / d_l
    zs, sg = np.zeros(len(Y)), np.zeros(len(Y))
    for v in range(n_v):
        for a in range(nm):
            o = coef_off[v][a]
            zs += r * np.abs(Y[:, o:o + 2 * art.q]).sum(1) * np.abs(art.basis[v, a]).max()
        sg += r * r * np.abs(Y[:, sig_off[v]:sig_off[v] + nm * nm]).sum(1)
    return EPS * (200 * (weights * zs + sg) + (cfg.t_trig + 2.0) * cfg.fs * slope * zs)


@pytest.mark.parametrize("n_det, n_modes, n_bands, q, sizes", [(1, 2, 2, 5, (1, 131, 4096, 4097)),
                                                              (3, 5, 4, 17, (1, 131))])
def test_outputs_to_lnl(n_det, n_modes, n_bands, q, sizes):
    cfg = wl.SMALL_BANDED.with_(name="banded_epilogue", sites=wl.SITES_HLV[:n_det], modes=wl.ALL_MODES[:n_modes],
                                n_bands=n_bands, n_nodes=60, q=q)
    inj = wl.injection_extrinsics(cfg)
    h = rbfl.Handle.from_config(cfg, wl.white_noise(cfg), inj)
    art = su.artefacts_from_exports(cfg, inj, **h.exports())
    m = 3 * max(sizes)
    idx, jit = wl.node_jitter(m, cfg.n_nodes, seed=q)
    qd = wl.queries(cfg, n=m, seed=q).near_nodes(h.nodes(), idx, jit)
    pool = np.ascontiguousarray(rbfl.params_soa(h, qd, cfg.t_trig))
    pool = pool[:, np.isfinite(run(h, pool))]         # inside the domain
    assert pool.shape[1] >= max(sizes)
    for n in sizes:
        P = pool[:, :n].copy()
        bad = sorted({n // 3, n - 1}) if n > 1 else []
        P[6, bad] = np.nan
        P[9, n // 2] += 10.0 if n > 1 else 0.0        # outside the window
        got, Y = run(h, P), run(h, P, what="interp")
        assert np.flatnonzero(np.isnan(got)).tolist() == bad and h.nan_count() == len(bad)
        keep = np.setdiff1d(np.unique(np.concatenate([np.arange(min(n, 131)), np.arange(max(0, n - 131), n)])), bad)
        p = P[:, keep]
        want = lk.meshfree_parts(art, p[0:4].T.copy(), p[4:9].T.copy(), p[9].copy(), p[10].copy(), Y=Y[keep])[0]
        fin = np.isfinite(want)
        assert np.array_equal(fin, np.isfinite(got[keep]))
        bound = rounding_bound(cfg, art, Y[keep], p[10])
        err = np.abs(got[keep][fin] - want[fin])
        print(f"[banded] {n_det} x {n_modes} x {n_bands}, n {n}: |ln L| <= {np.abs(want[fin]).max():.3g}, max |d| "
              f"{err.max():.2e}, bound from {bound.min():.2e}", flush=True)
        assert (err <= bound[fin]).all() and fin.sum() >= len(keep) - 1
