"""Batch sizes at which the online stage changes kernels: every batch gives
each proposal the interpolated outputs and ln L of a large batch."""
import numpy as np
import pytest

from paper_2508_04172_amd import rbfl
from paper_2508_04172_amd import workloads as wl

pytestmark = pytest.mark.gpu

N_ALL = 110_000


@pytest.fixture(scope="module")
def case():
    """A handle of 256 padded columns, N_ALL proposals, and their outputs and ln L
    from one large batch (the 64 x 128 tile, 16 proposals per epilogue workgroup)."""
    import torch
    cfg = wl.SMALL_MULTI.with_(name="batch_sizes", n_nodes=60, q=12)
    h = rbfl.Handle.from_config(cfg, wl.white_noise(cfg), wl.injection_extrinsics(cfg))
    idx, jit = wl.node_jitter(N_ALL, cfg.n_nodes)
    qd = wl.queries(cfg, n=N_ALL).near_nodes(h.nodes(), idx, jit)
    p = torch.from_numpy(rbfl.params_soa(h, qd, cfg.t_trig)).cuda()
    h.reserve(N_ALL)
    return h, p, interp(h, p), lnl(h, p)


def interp(h, p):
    import torch
    out = torch.empty(p.shape[1], h.sizes()["K"], device="cuda", dtype=torch.float64)
    h.interp(p.data_ptr(), p.shape[1], out.data_ptr(), rbfl.FORM_FP64, torch.cuda.current_stream().cuda_stream)
    return out


def lnl(h, p):
    import torch
    out = torch.empty(p.shape[1], device="cuda", dtype=torch.float64)
    h.eval(p.data_ptr(), p.shape[1], out.data_ptr(), rbfl.FORM_FP64, torch.cuda.current_stream().cuda_stream)
    return out.cpu().numpy()


# 256 columns are 8 tiles of 32: the tiles change at 2880 / 8 and 22000 / 8 rows
# of 32 proposals, the epilogue at 4096 proposals; remainders of 16, 32 and 64.
# Up to 1024 proposals (64 groups of at most 16) ln L is one launch.
@pytest.mark.parametrize("n", [1, 2, 15, 17, 33, 63, 65, 1021, 1024, 1025, 4096, 4097, 11487, 11489, 12289, 65505, 87967, 87969])
def test_batch_size(case, n):
    import torch
    h, p, ref, ref_lnl = case
    cols = slice(N_ALL - n, N_ALL)                    # the tail: other tile positions than in the large batch
    sub = p[:, cols].contiguous()
    # the same MFMA over the same rows in the same order: the outputs agree bit for bit
    assert torch.equal(interp(h, sub), ref[cols])
    got, want = lnl(h, sub), ref_lnl[cols]
    fin = np.isfinite(want)
    assert np.array_equal(fin, np.isfinite(got)) and np.array_equal(np.isnan(want), np.isnan(got))
    # the epilogue sums fewer than 300 products per proposal, each below 1e5 here
    # (SNR 20, distances from half the injection's): 300 eps 1e5 < 1e-8
    assert fin.sum() == 0 or np.abs(got[fin] - want[fin]).max() <= 1e-8


# up to 4096 proposals the epilogue counts the NaN results itself, one slot each
@pytest.mark.parametrize("n", [1, 5, 4096, 4097])
def test_nan_count(case, n):
    h, p, _, _ = case
    sub = p[:, :n].contiguous()
    lnl(h, sub)
    assert h.nan_count() == 0
    bad = sorted({0, n // 2, n - 1})
    sub[8, bad] = float("nan")
    assert np.flatnonzero(np.isnan(lnl(h, sub))).tolist() == bad
    assert h.nan_count() == len(bad)


# 2 column tiles of 128: rounds of 128 (256 x 128) and 256 (128 x 128) tiles along
# the proposals; 90,000 are 2.75 and 2.75 of them, 100,000 3.06, 110,000 3.36
@pytest.mark.parametrize("n", [90_000, 99_999, N_ALL])
@pytest.mark.parametrize("v", range(7))
def test_large_tiles_agree(case, v, n):
    """Each large tile past the smaller tiles' range, with and without a short
    last round that these take over."""
    import torch
    h, p, ref, _ = case
    h.set_variant(rbfl.FORM_FP64, v)
    try:
        assert torch.equal(interp(h, p[:, :n].contiguous()), ref[:n])
    finally:
        h.set_variant(rbfl.FORM_FP64, 0)


# two events of 243 and 19 columns: 8 and 1 tiles of 32 per 32 proposals, so the
# plan's tiles change at 2880 and 22000 of them, the epilogue at 8192 and 16,384
# proposals
@pytest.mark.parametrize("counts", [(1, 1), (33, 700), (8191, 1), (8192, 1), (11_489, 1), (8000, 8191), (60_000, 9000), (100_001, 60_000)])
def test_plan_sizes(case, counts):
    """A two-event plan at sizes on both sides of its tile changes, every rows +
    GEMM variant pinned, against the per-event evaluation."""
    import torch
    h, p, _, _ = case
    cfg = wl.CFG1.with_(name="plan_sizes", seg_len=8.0, n_nodes=45, q=9)
    h2 = rbfl.Handle.from_config(cfg, wl.white_noise(cfg), wl.injection_extrinsics(cfg))
    idx, jit = wl.node_jitter(counts[1], cfg.n_nodes)
    qd = wl.queries(cfg, n=counts[1]).near_nodes(h2.nodes(), idx, jit)
    p2 = torch.from_numpy(rbfl.params_soa(h2, qd, cfg.t_trig)).cuda()
    p1 = p[:, :counts[0]].contiguous()
    want = np.concatenate([lnl(h, p1), lnl(h2, p2)])
    both = torch.cat([p1, p2], dim=1).contiguous()
    out = torch.empty(sum(counts), device="cuda", dtype=torch.float64)
    st = torch.cuda.current_stream().cuda_stream
    plan = rbfl.Plan([h, h2], counts, both.data_ptr(), out.data_ptr(), rbfl.PLAN_GRAPH, st)
    for v in (3, 4, 5):
        plan.set_variant(v, st)
        for replay in range(2):
            out.fill_(7.0)
            plan.launch(st)
            got = out.cpu().numpy()
            fin = np.isfinite(want)
            assert np.array_equal(fin, np.isfinite(got)), f"variant {v}"
            # the bound of the other multi-event tests: the same products, summed by another kernel
            assert np.abs(got[fin] - want[fin]).max(initial=0.0) <= 1e-12 * max(1.0, np.abs(want[fin]).max(initial=0.0))


# one column tile (128): the contraction forms its own rows from 12288 proposals on
# with few rows, from 32768 on with more than 512, except for a last partial round
# of less than 8192 past each 49152
@pytest.mark.parametrize("nodes, n", [(45, 12287), (45, 12288), (45, 12351), (45, 49152), (45, 49153), (45, 57343),
                                      (45, 57345), (500, 12289), (600, 32767), (600, 32769), (600, 49217)])
def test_one_column_tile(nodes, n):
    """Batches on both sides of the rule against the same proposals in slices
    below it: the same row values and MFMA order, so the same bits."""
    import torch
    cfg = wl.CFG1.with_(name="one_tile", seg_len=8.0, n_nodes=nodes, q=9, poly_degree=3)
    h = rbfl.Handle.from_config(cfg, wl.white_noise(cfg), wl.injection_extrinsics(cfg))
    idx, jit = wl.node_jitter(n, cfg.n_nodes)
    qd = wl.queries(cfg, n=n).near_nodes(h.nodes(), idx, jit)
    p = torch.from_numpy(rbfl.params_soa(h, qd, cfg.t_trig)).cuda()
    h.reserve(n)
    got = interp(h, p)
    for b in range(0, n, 8192):
        assert torch.equal(interp(h, p[:, b:b + 8192].contiguous()), got[b:b + 8192])


# column counts around multiples of 32 and 64: tiles of padding columns are left out
@pytest.mark.parametrize("q", [15, 16, 31, 32, 47, 48, 60])
def test_column_counts(q):
    import torch
    cfg = wl.CFG1.with_(name="columns", seg_len=8.0, n_nodes=100, q=q)
    h = rbfl.Handle.from_config(cfg, wl.white_noise(cfg), wl.injection_extrinsics(cfg))
    n = 20_000                                        # forms its own rows
    idx, jit = wl.node_jitter(n, cfg.n_nodes)
    qd = wl.queries(cfg, n=n).near_nodes(h.nodes(), idx, jit)
    p = torch.from_numpy(rbfl.params_soa(h, qd, cfg.t_trig)).cuda()
    h.reserve(n)
    got = interp(h, p)
    # every output of one proposal is the weighted sum of its row (K = 2 q + 1
    # sums of 105 products): against torch with the library's nodes and weights
    x = (p[:4].T / torch.from_numpy(h.frame()["semi"].copy()).cuda())[:256]
    nodes, W = torch.from_numpy(h.nodes()).cuda(), torch.from_numpy(h.weights()).cuda()
    d2 = ((x[:, None, :] - nodes[None]) ** 2).sum(-1)
    phi = torch.cat([torch.exp(-h.eps() ** 2 * d2), torch.ones(256, 1, device="cuda", dtype=torch.float64), x], 1)
    assert got.shape[1] == 2 * q + 1 and W.shape == (105, 2 * q + 1)
    bound = 105 * 8 * 2.2e-16 * (phi.abs() @ W.abs())  # rows to a few units, sums of 105 terms in any order
    assert ((got[:256] - phi @ W).abs() <= bound).all()
    for step in (8192, 700):                          # the other tiles: the same bits
        for b in range(0, n, step):
            assert torch.equal(interp(h, p[:, b:b + step].contiguous()), got[b:b + step])


# one launch against the staged kernels (which the stage timers keep): 1 to 16
# proposals per workgroup, one and seven tiles of 64 columns, ragged last groups,
# and the sizes around the largest that takes one launch
@pytest.mark.parametrize("sites, modes, nodes, degree, q, sizes", [
    (1, 1, 60, 1, 5, [1, 2, 255, 256, 257, 1000, 2049, 4081, 4096, 4097]),
    (1, 2, 150, 3, 13, [1, 3, 65, 511]),
    (3, 4, 300, 2, 16, [1, 31, 36, 37, 100, 255, 289, 575, 576, 577]),
])
def test_one_launch(sites, modes, nodes, degree, q, sizes):
    import torch
    cfg = wl.SMALL_MULTI.with_(name="one_launch", sites=wl.SITES_HLV[:sites], modes=wl.ALL_MODES[:modes], n_nodes=nodes,
                               poly_degree=degree, q=q, eps=0.0)
    h = rbfl.Handle.from_config(cfg, wl.white_noise(cfg), wl.injection_extrinsics(cfg))
    n_all = max(sizes)
    idx, jit = wl.node_jitter(n_all, cfg.n_nodes)
    qd = wl.queries(cfg, n=n_all).near_nodes(h.nodes(), idx, jit)
    P = np.ascontiguousarray(rbfl.params_soa(h, qd, cfg.t_trig))
    P[9, ::7] = cfg.t_trig + 10.0                     # outside the window
    P[6, ::11] = np.nan
    p = torch.from_numpy(P).cuda()
    h.reserve(n_all)
    for n in sizes:
        sub = p[:, n_all - n:].contiguous()
        h.profile(True)
        want = lnl(h, sub)
        h.profile(False)
        for _ in range(2):                            # the second finds the counters that the first left
            assert np.array_equal(lnl(h, sub), want, equal_nan=True)
            assert h.nan_count() == int(np.isnan(want).sum())


# split form, 256 columns: 32 x 32 tiles up to 1024 of them (4096 proposals), four
# rows per thread up to 2^20 row values (10,922 proposals of 96 rows)
@pytest.mark.parametrize("v, sizes", [(2, [1, 31, 32, 33, 1021, 4096, 4097, 10_922, 10_923]), (0, [1, 100]),
                                      (1, [33, 700]), (3, [17, 4096])])
def test_split_batch_size(case, v, sizes):
    import torch
    h, p, _, _ = case
    stream = torch.cuda.current_stream().cuda_stream
    n_all = 20_000

    def run(sub):
        n = sub.shape[1]
        out = torch.empty(n, h.sizes()["K"], device="cuda", dtype=torch.float64)
        l = torch.empty(n, device="cuda", dtype=torch.float64)
        h.interp(sub.data_ptr(), n, out.data_ptr(), rbfl.FORM_SPLIT, stream)
        h.eval(sub.data_ptr(), n, l.data_ptr(), rbfl.FORM_SPLIT, stream)
        return out, l.cpu().numpy()

    h.prepare(rbfl.FORM_SPLIT)
    h.set_variant(rbfl.FORM_SPLIT, v)
    ref, ref_lnl = run(p[:, :n_all].contiguous())
    for n in sizes:
        got, got_lnl = run(p[:, n_all - n:n_all].contiguous())
        # integer sums, combined alike: the outputs agree bit for bit; ln L as in test_batch_size
        assert torch.equal(got, ref[n_all - n:])
        want = ref_lnl[n_all - n:]
        fin = np.isfinite(want)
        assert np.array_equal(fin, np.isfinite(got_lnl))
        assert fin.sum() == 0 or np.abs(got_lnl[fin] - want[fin]).max() <= 1e-8
