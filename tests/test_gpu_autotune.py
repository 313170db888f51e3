"""The tile autotuner on batches that do not run the tile variants: each variant's
time is that of its own tile, and the handle keeps the tile that it had.

The times follow from the tiles' chains: for one tile of few proposals the 16
products per row step of a wave of the 256 x 128 tile take four times as long as
the 4 of the 64 x 64 tile (64 cycles each; 605 rows: about 65 against 16 us beside
the rows' 6 to 10), and the 8 of a 64 x 128 tile eight times as long as the one of
the 32 x 32 tile that a small plan runs."""
import numpy as np
import pytest

from paper_2508_04172_amd import rbfl
from paper_2508_04172_amd import workloads as wl

pytestmark = pytest.mark.gpu


def setup(cfg, n):
    import torch
    h = rbfl.Handle.from_config(cfg, wl.white_noise(cfg), wl.injection_extrinsics(cfg))
    idx, jit = wl.node_jitter(n, cfg.n_nodes)
    qd = wl.queries(cfg, n=n).near_nodes(h.nodes(), idx, jit)
    return h, torch.from_numpy(rbfl.params_soa(h, qd, cfg.t_trig)).cuda()


def stream():
    import torch
    return torch.cuda.current_stream().cuda_stream


@pytest.mark.parametrize("before", [0, 3, 6])
def test_small_batch_keeps_the_tile(before):
    cfg = wl.SMALL_MULTI.with_(name="autotune", n_nodes=600, q=12, eps=0.0)
    n = 64
    h, p = setup(cfg, n)
    h.reserve(n)
    h.set_variant(rbfl.FORM_FP64, before)
    tunes = [h.autotune(p.data_ptr(), n, rbfl.FORM_FP64, stream()) for _ in range(3)]
    print(f"[autotune] {n} proposals, tile {before} before: {tunes[0]}", flush=True)
    assert all(t["variant"] == before and len(t["ms"]) == rbfl_variants() for t in tunes)
    best = np.min([t["ms"] for t in tunes], axis=0)   # one launch each: the least disturbed
    assert best[5] >= 1.5 * best[4]


def rbfl_variants():
    return int(rbfl.load().rbfl_variants(rbfl.FORM_FP64))


def test_one_column_tile_keeps_the_tile():
    """Up to 128 outputs a batch of this size forms its own rows (the fused variant,
    which the tuner may still prefer to that, is the last one)."""
    cfg = wl.CFG1.with_(name="autotune_one", seg_len=8.0, n_nodes=200, q=20, eps=0.0)
    n = 20_000
    h, p = setup(cfg, n)
    h.reserve(n)
    h.set_variant(rbfl.FORM_FP64, 2)
    tune = h.autotune(p.data_ptr(), n, rbfl.FORM_FP64, stream())
    print(f"[autotune] {n} proposals, one column tile: {tune}", flush=True)
    assert tune["variant"] in (2, rbfl_variants() - 1) and len(tune["ms"]) == rbfl_variants()


def test_small_plan_times_the_tiles():
    import torch
    cfg = wl.SMALL_MULTI.with_(name="autotune_plan", n_nodes=1000, q=12, eps=0.0)
    n = 64
    h, p = setup(cfg, 2 * n)
    out = torch.empty(2 * n, dtype=torch.float64, device="cuda")
    plan = rbfl.Plan([h, h], [n, n], p.data_ptr(), out.data_ptr(), rbfl.PLAN_AUTOTUNE, stream())
    info = plan.info()
    times = []
    for _ in range(7):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        plan.launch(stream())
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    print(f"[autotune] plan {info}, ms per launch {np.median(times):.4f}", flush=True)
    assert info["variant"] == 3 and len(info["tune_ms"]) == 6
    assert min(info["tune_ms"][3:]) >= 1.3 * np.median(times)
    # the tiles' bits do not differ: the same ln L with every variant pinned
    ref = out.cpu().numpy()
    for v in (3, 4, 5):
        plan.set_variant(v, stream())
        out.fill_(7.0)
        plan.launch(stream())
        assert np.array_equal(out.cpu().numpy(), ref, equal_nan=True)
