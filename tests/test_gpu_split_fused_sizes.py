"""The split form with ln L finished inside its contraction, at batch sizes on both
sides of the rule that leaves out its column tiles of padding, against the separate
epilogue."""
import numpy as np
import pytest

from paper_2508_04172_amd import rbfl
from paper_2508_04172_amd import workloads as wl

pytestmark = pytest.mark.gpu


# 41 of 128 padded columns: two column tiles of 64, one of them padding, both run
# up to 256 tiles (128 proposal tiles of 128 proposals); 165 of 256: four, one padding
@pytest.mark.parametrize("sites, modes, q, sizes", [(1, 1, 20, [1, 129, 16_384, 16_385]), (3, 1, 27, [8192, 8193])])
def test_fused_split_matches_separate(sites, modes, q, sizes):
    import torch
    cfg = wl.SMALL_MULTI.with_(name="split_fused", sites=wl.SITES_HLV[:sites], modes=wl.ALL_MODES[:modes],
                               n_nodes=100, q=q, eps=0.0)
    h = rbfl.Handle.from_config(cfg, wl.white_noise(cfg), wl.injection_extrinsics(cfg))
    n_all = max(sizes)
    idx, jit = wl.node_jitter(n_all, cfg.n_nodes)
    qd = wl.queries(cfg, n=n_all).near_nodes(h.nodes(), idx, jit)
    p = torch.from_numpy(rbfl.params_soa(h, qd, cfg.t_trig)).cuda()
    h.prepare(rbfl.FORM_SPLIT)
    h.reserve(n_all)
    stream = torch.cuda.current_stream().cuda_stream

    def lnl(sub, fused):
        h.fuse_epilogue(False, split=fused)
        out = torch.full((sub.shape[1],), 7.0, device="cuda", dtype=torch.float64)
        h.eval(sub.data_ptr(), sub.shape[1], out.data_ptr(), rbfl.FORM_SPLIT, stream)
        return out.cpu().numpy()

    ref = lnl(p, True)
    for n in sizes:
        sub = p[:, n_all - n:].contiguous()
        got, want = lnl(sub, True), lnl(sub, False)
        assert np.array_equal(got, ref[n_all - n:], equal_nan=True)        # every batch the same bits
        fin = np.isfinite(want)
        assert np.array_equal(fin, np.isfinite(got))
        # the same fewer than 300 products, each below 1e5 here, summed in another
        # order: 300 eps 1e5 < 1e-8
        assert fin.sum() == 0 or np.abs(got[fin] - want[fin]).max() <= 1e-8
