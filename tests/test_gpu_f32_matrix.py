"""The fp32 scan on the fp32 matrix units (trees of at most 64 nodes, dstate 64 / 128 / 256): tile edges and
remainders in nodes and headdim against the oracle, and against the plain FMA kernel, whose fp32 sums it forms in
another order (2 S + N terms each: S = 256, N = 64 leaves 2^-24 * sqrt(576) < 2e-6 of the rms, and expf's argument
error 6e-8 |s| on either side; asserted 2e-5)."""
import numpy as np
import pytest

from paper_2505_14969_amd import synth
from helpers import TOL, assert_parity, to_dev, to_host
from test_gpu_parity import _rand, st  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,H,P,S,G,with_h0", [(1, 2, 64, 64, 1, True), (31, 3, 33, 128, 1, True), (32, 2, 31, 128, 1, False),
                                               (33, 2, 64, 128, 2, True), (63, 4, 1, 64, 1, True), (64, 2, 100, 256, 1, True),
                                               (7, 130, 64, 128, 1, True), (1, 2, 65, 128, 1, False),
                                               (2, 2, 96, 64, 1, False), (3, 2, 96, 64, 1, False), (3, 2, 128, 64, 1, False), (4, 2, 129, 64, 1, False),
                                               (5, 2, 256, 64, 1, False)])
def test_f32_scan_tiles(st, oracle, N, H, P, S, G, with_h0):
    B = 2
    g = np.random.default_rng(N)
    par = np.stack([synth.gen_tree(N, min(N - 1, 4), 4, g) if N > 1 else np.array([-1]), synth.chain_tree(N)]).astype(np.int32)
    x, dt, A, Bm, Cm, D, h0 = _rand(40 + N, "f32", B, N, H, P, S, G, h0=with_h0)
    want = oracle.ssd_paths(par, x, dt, A, Bm, Cm, D, h0)
    args = (to_dev(par), to_dev(x), to_dev(dt), to_dev(A), to_dev(Bm), to_dev(Cm), to_dev(D), to_dev(h0))
    y = to_host(st.stree_tree_ssd(*args))
    assert_parity(y, want, TOL["f32"], "y", kind="y")
    assert_parity(y, to_host(st.stree_tree_ssd(*args, force_fma=True)), 2e-5, "y against the FMA kernel", kind="y")


@pytest.mark.parametrize("N,P,S,G", [(64, 64, 128, 1), (33, 40, 64, 2), (20, 65, 256, 1)])
def test_f32_scan_reports_bad_trees(st, oracle, N, P, S, G):
    """A bad parent in either row block: that sequence's y is zero in all rows and columns and its status names the
    node; the others are untouched."""
    import torch
    B, H = 4, 2
    par = np.stack([synth.gen_tree(N, 5, 4, np.random.default_rng(b)) for b in range(B)]).astype(np.int32)
    par[1, 4], par[3, N - 1] = 4, N + 7
    x, dt, A, Bm, Cm, D, h0 = _rand(60 + N, "f32", B, N, H, P, S, G)
    status = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    out = torch.full((B, N, H, P), 3.0, device="cuda")
    got = to_host(st.stree_tree_ssd(to_dev(par), to_dev(x), to_dev(dt), to_dev(A), to_dev(Bm), to_dev(Cm), to_dev(D),
                                    to_dev(h0), out=out, status=status))
    assert list(to_host(status)) == [0, 5, 0, N]
    assert not got[1].any() and not got[3].any()
    keep = [0, 2]
    want = oracle.ssd_paths(par[keep], x[keep], dt[keep], A, Bm[keep], Cm[keep], D, h0[keep])
    assert_parity(got[keep], want, TOL["f32"], "sequences beside the bad ones", kind="y")


@pytest.mark.parametrize("N,P,bad", [(15, 64, 3), (15, 64, 14), (33, 33, 7), (33, 33, 32), (64, 40, 20), (64, 40, 45)])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_f32_scan_keeps_a_bad_node_to_its_descendants(st, oracle, N, P, bad, value):
    """x of one node is not finite (all its values, or one of them; in the second sequence its weight is 0 as well): the
    rows that do not descend from it are what the oracle gives, and the others are the FMA kernel's, which skips
    products with a weight of 0."""
    B, H, S, G = 3, 2, 64, 1
    par = np.stack([synth.full_binary_tree(7)[:N]] * B).astype(np.int32)
    x, dt, A, Bm, Cm, D, h0 = _rand(70 + N, "f32", B, N, H, P, S, G)
    dt[1, bad] = 0.0
    spoilt = x.copy()
    spoilt[0, bad], spoilt[1, bad], spoilt[2, bad, 1, P - 1] = value, value, value
    want = oracle.ssd_paths(par, x, dt, A, Bm, Cm, D, h0)
    below = np.array([bad in _path(par[0], i) for i in range(N)])
    for h in (h0, None):
        args = [to_dev(a) for a in (par, spoilt, dt, A, Bm, Cm, D, h)]
        got, fma = to_host(st.stree_tree_ssd(*args)), to_host(st.stree_tree_ssd(*args, force_fma=True))
        assert np.isfinite(got[:, ~below]).all() and np.isfinite(got[2, :, 0]).all() and np.isfinite(got[2, :, 1, :P - 1]).all()
        assert np.isfinite(got[1, np.arange(N) != bad]).all()
        if h is not None:
            assert_parity(got[:, ~below], want[:, ~below], TOL["f32"], "rows beside the bad node", kind="y")
        ok = np.isfinite(fma)
        assert np.array_equal(np.isfinite(got), ok) and np.array_equal(np.isnan(got), np.isnan(fma))
        assert np.array_equal(got[~ok & ~np.isnan(fma)], fma[~ok & ~np.isnan(fma)])           # infinities by sign
        assert_parity(np.where(ok, got, 0), np.where(ok, fma, 0), 2e-5, "finite rows against the FMA kernel", kind="y")


def _path(parent, i):
    while i >= 0:
        yield i
        i = parent[i]


def test_f32_scan_of_more_heads_than_one_grid_dimension_holds(st):
    """1025 x 65535 heads of one column, one node: as one wave each, 2^32 work items and more in one grid dimension."""
    import torch
    B, N, H, P, S, G = 1025, 1, 65535, 1, 64, 1
    gen = torch.Generator(device="cuda").manual_seed(3)
    rand = lambda *s: torch.randn(s, generator=gen, device="cuda")  # noqa: E731
    x, dt, Bm, Cm, A, D = rand(B, N, H, P), rand(B, N, H).abs(), rand(B, N, G, S), rand(B, N, G, S), -rand(H).abs(), rand(H)
    y = st.stree_tree_ssd(torch.full((B, N), -1, dtype=torch.int32, device="cuda"), x, dt, A, Bm, Cm, D)
    want = ((Bm * Cm).sum(-1) * dt + D).unsqueeze(-1) * x
    # one product of 64 fp32 terms each, in another order
    assert bool(((y - want).abs() <= 2e-5 * (want.abs() + x.abs() * (dt * 8 + 1).unsqueeze(-1))).all())
