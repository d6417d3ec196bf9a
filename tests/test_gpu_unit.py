"""GPU parity of the tree scan (and replay + scan) of at most 64 nodes, a workgroup per head: remainders of the 32-node
blocks, every head shape and state type, paths longer than the rows held at once, and both sides of the lines between its
forms and the persistent kernel."""
import numpy as np
import pytest

from paper_2505_14969_amd import synth
from helpers import TOL, assert_parity, to_dev, to_host
from test_gpu_parity import _rand, _run_ssd, _trees, st  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

SHAPES = [(64, 128, 1), (64, 64, 2), (64, 256, 1), (128, 128, 2)]


@pytest.mark.parametrize("N", [1, 2, 31, 32, 33, 63, 64])
@pytest.mark.parametrize("P,S,G", SHAPES)
def test_unit_kernel_block_remainders(st, oracle, N, P, S, G):
    B, H = 3, 4
    parent = _trees(140 + N, B, N)
    parent[0] = synth.chain_tree(N)
    x, dt, A, Bm, Cm, D, h0 = _rand(141 + N, "bf16", B, N, H, P, S, G)
    A[0], A[1] = -0.05, -60.0                            # weights by factors and by an exponential per pair
    dt[2, N // 2] = 0.0
    if N == 1:
        D = None        # (one row: dt <C, B> + D may cancel, and nothing else sets the scale that errors are measured by)
    for state in (h0, None):
        want = oracle.ssd_paths(parent, x, dt, A, Bm, Cm, D, state)
        got = _run_ssd(st, "bf16", parent, x, dt, A, Bm, Cm, D, state)
        assert_parity(got, want, TOL["bf16"], f"unit kernel N={N} P={P} S={S} state={state is not None}", kind="y")
    rounded = synth.round_to_bf16(h0)
    y = st.stree_tree_ssd(to_dev(parent), to_dev(x, "bf16"), to_dev(dt), to_dev(A), to_dev(Bm, "bf16"), to_dev(Cm, "bf16"),
                          to_dev(D), to_dev(rounded, "bf16"))
    assert np.array_equal(to_host(y), _run_ssd(st, "bf16", parent, x, dt, A, Bm, Cm, D, rounded))


def _replay(st, oracle, B, N, Np, H, P, S, G, state, seed):
    import torch
    parent, pparent = _trees(seed, B, N), _trees(seed + 1, B, Np)
    pparent[0] = synth.chain_tree(Np)
    x, dt, A, Bm, Cm, D, h0 = _rand(seed + 2, "bf16", B, N, H, P, S, G)
    px, pdt, _, pB, _, _, _ = _rand(seed + 3, "bf16", B, Np, H, P, S, G)
    if state == "bf16":
        h0 = synth.round_to_bf16(h0)
    acc = np.arange(B, dtype=np.int32) * 7 % Np
    acc[0], acc[1], acc[2] = Np - 1, -1, Np
    kept = np.where(acc >= Np, -1, acc).astype(np.int32)
    want_h, _ = oracle.commit(pparent, kept, px, pdt, A, pB, h0)
    h_in = to_dev(h0, "bf16") if state == "bf16" else to_dev(h0)
    rstatus = to_dev(np.full(B, 9, dtype=np.int32))
    args = (to_dev(pparent), to_dev(acc), to_dev(px, "bf16"), to_dev(pdt), to_dev(pB, "bf16"), to_dev(parent), to_dev(x, "bf16"),
            to_dev(dt), to_dev(A), to_dev(Bm, "bf16"), to_dev(Cm, "bf16"), to_dev(D))
    y, h = st.stree_tree_ssd_replay(*args, h_in, replay_status=rstatus)
    assert to_host(rstatus).tolist() == [0, 0, -1] + [0] * (B - 3)
    got_h = to_host(h)
    assert np.array_equal(got_h[1], h0[1]) and np.array_equal(got_h[2], h0[2])
    if state == "bf16":
        assert np.all(np.abs(got_h - want_h) <= 2.0 ** -8 * np.abs(want_h) + 1e-4 * np.abs(want_h).max())
        want_h = got_h.astype(np.float64)
    else:
        assert_parity(got_h, want_h, 1e-4, f"replayed state N={N} Np={Np} P={P} S={S}", kind="state")
    want_y = oracle.ssd_paths(parent, x, dt, A, Bm, Cm, D, want_h)
    assert_parity(to_host(y), want_y, TOL["bf16"], f"scan behind the replay N={N} Np={Np} P={P} S={S}", kind="y")
    y2, _ = st.stree_tree_ssd_replay(*args, h_in, h_out=h_in)
    assert torch.equal(y2, y) and torch.equal(h_in, h)


@pytest.mark.parametrize("N,Np", [(1, 1), (32, 33), (33, 15), (40, 16), (64, 64), (5, 31)])
@pytest.mark.parametrize("P,S,G", SHAPES)
@pytest.mark.parametrize("state", ["f32", "bf16"])
def test_unit_kernel_replay(st, oracle, N, Np, P, S, G, state):
    _replay(st, oracle, 6, N, Np, 2, P, S, G, state, 160 + N + Np)


# the state requested late (more heads than are resident at once), and the persistent kernel's band on either side
@pytest.mark.parametrize("B,N,H,P,S,state", [(89, 34, 16, 64, 64, "f32"), (89, 33, 16, 64, 64, "bf16"), (88, 33, 16, 64, 128, "f32"),
                                             (41, 33, 16, 64, 128, "f32"), (40, 33, 16, 64, 128, "f32"), (41, 32, 16, 64, 128, "f32"),
                                             (89, 33, 16, 64, 128, "f32"), (89, 20, 16, 64, 128, "bf16"), (90, 20, 8, 128, 128, "f32"),
                                             (65, 41, 16, 64, 128, "bf16"), (65, 40, 16, 64, 128, "bf16"), (79, 64, 16, 64, 128, "bf16"),
                                             (80, 64, 16, 64, 128, "bf16"), (33, 55, 16, 64, 128, "f32"), (33, 54, 16, 64, 128, "f32"),
                                             (41, 53, 16, 64, 128, "f32"), (93, 49, 16, 64, 128, "f32"), (92, 49, 16, 64, 128, "f32"),
                                             (49, 37, 8, 128, 128, "f32"), (48, 41, 8, 128, 128, "f32"), (64, 64, 8, 128, 128, "f32"),
                                             (65, 64, 8, 128, 128, "f32"), (64, 36, 8, 128, 128, "f32"), (49, 60, 8, 128, 128, "bf16"), (89, 32, 16, 64, 64, "f32"),
                                             (89, 33, 16, 64, 256, "f32"), (89, 33, 16, 64, 256, "bf16"), (89, 33, 8, 128, 128, "bf16"),
                                             (90, 34, 8, 128, 128, "f32")])
def test_unit_kernel_replay_at_the_lines_between_its_forms(st, oracle, B, N, H, P, S, state):
    _replay(st, oracle, B, N, 21, H, P, S, 1, state, 190 + B + N)


def test_persistent_replay_of_several_groups(st, oracle):
    """Runs of two and three heads that cross groups and sequences (512 workgroups for 1072 heads in 4 groups)."""
    _replay(st, oracle, 67, 60, 21, 16, 64, 128, 4, "f32", 990)


@pytest.mark.parametrize("B,N,H,S", [(65, 49, 16, 128), (64, 49, 16, 128), (65, 48, 16, 128), (106, 50, 16, 64), (107, 50, 16, 64),
                                       (49, 57, 16, 128), (49, 56, 16, 128), (81, 45, 16, 128), (81, 44, 16, 128), (69, 57, 16, 64)])
def test_unit_kernel_scan_at_the_lines_between_its_forms(st, oracle, B, N, H, S):
    parent = _trees(230 + B, B, N)
    x, dt, A, Bm, Cm, D, h0 = _rand(231 + B, "bf16", B, N, H, 64, S, 1)
    want = oracle.ssd_paths(parent, x, dt, A, Bm, Cm, D, h0)
    assert_parity(_run_ssd(st, "bf16", parent, x, dt, A, Bm, Cm, D, h0), want, TOL["bf16"], f"scan B={B} N={N} S={S}", kind="y")


@pytest.mark.parametrize("B,N,H", [(65, 57, 16), (65, 56, 16), (80, 64, 16), (81, 64, 16), (65, 53, 16), (65, 52, 16), (81, 59, 16), (81, 58, 16),
                                   (165, 61, 16)])
def test_scan_of_a_bf16_state_at_the_lines_between_its_forms(st, oracle, B, N, H):
    parent = _trees(260 + B, B, N)
    x, dt, A, Bm, Cm, D, h0 = _rand(261 + B + N, "bf16", B, N, H, 64, 128, 1)
    h0 = synth.round_to_bf16(h0)
    want = oracle.ssd_paths(parent, x, dt, A, Bm, Cm, D, h0)
    y = st.stree_tree_ssd(to_dev(parent), to_dev(x, "bf16"), to_dev(dt), to_dev(A), to_dev(Bm, "bf16"), to_dev(Cm, "bf16"),
                          to_dev(D), to_dev(h0, "bf16"))
    assert_parity(to_host(y), want, TOL["bf16"], f"scan of a bf16 state B={B} N={N}", kind="y")


@pytest.mark.parametrize("P,S,G", SHAPES)
def test_few_nodes_with_huge_token_strides(st, oracle, P, S, G):
    """Rows 256 MiB apart, NaN between them: sixteen rows on, a 32-bit byte offset is back between the tree's rows (and a
    weight of 0 does not undo a NaN)."""
    import torch
    B, N, H, stride = 1, 3, 2, (1 << 27) + 64
    parent, pparent = _trees(180, B, N), _trees(181, B, 5)
    x, dt, A, Bm, Cm, D, h0 = _rand(182, "bf16", B, N, H, P, S, G)
    px, pdt, _, pB, _, _, _ = _rand(183, "bf16", B, 5, H, P, S, G)
    room = torch.full((N * stride,), float("nan"), dtype=torch.bfloat16, device="cuda").view(1, N, stride)
    views = []
    for k, a in enumerate((x, Bm, Cm)):
        rows = room[:, :, 4096 * k:4096 * k + a.shape[2] * a.shape[3]]
        rows.copy_(to_dev(a, "bf16").reshape(1, N, -1))
        views.append(rows.unflatten(2, a.shape[2:]))
    now = (to_dev(parent), views[0], to_dev(dt), to_dev(A), views[1], views[2], to_dev(D), to_dev(h0))
    want = oracle.ssd_paths(parent, x, dt, A, Bm, Cm, D, h0)
    assert_parity(to_host(st.stree_tree_ssd(*now)), want, TOL["bf16"], "scan", kind="y")
    acc = np.array([4], dtype=np.int32)
    want_h, _ = oracle.commit(pparent, acc, px, pdt, A, pB, h0)
    y, h = st.stree_tree_ssd_replay(to_dev(pparent), to_dev(acc), to_dev(px, "bf16"), to_dev(pdt), to_dev(pB, "bf16"), *now)
    assert_parity(to_host(h), want_h, 1e-4, "replayed state", kind="state")
    assert_parity(to_host(y), oracle.ssd_paths(parent, x, dt, A, Bm, Cm, D, want_h), TOL["bf16"], "scan behind the replay", kind="y")
