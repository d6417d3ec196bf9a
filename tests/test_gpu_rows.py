"""GPU parity of the tree scan of 65 .. 256 nodes, a workgroup per head whose waves own 32 nodes each: remainders of node
blocks and phases, both forms of the decay weights side by side, every head shape and state type."""
import numpy as np
import pytest

from paper_2505_14969_amd import synth
from helpers import TOL, assert_parity, to_dev, to_host
from test_gpu_parity import _rand, _run_ssd, _trees, st  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [65, 96, 97, 128, 129, 160, 161, 193, 224, 225, 256])
@pytest.mark.parametrize("P,S,G", [(64, 128, 1), (64, 64, 2), (64, 256, 1), (128, 128, 2)])
def test_rows_kernel_block_remainders(st, oracle, N, P, S, G):
    B, H = 3, 4
    parent = _trees(40 + N, B, N)
    parent[0] = synth.chain_tree(N)
    x, dt, A, Bm, Cm, D, h0 = _rand(41 + N, "bf16", B, N, H, P, S, G)
    # weights by a factor per row and one per column (weak decays), by an exponential per pair (strong ones), and a
    # head that is on either side of the line by the sequence
    A[0], A[1], A[2] = -0.05, -60.0, -2.0
    want = oracle.ssd_paths(parent, x, dt, A, Bm, Cm, D, h0)
    got = _run_ssd(st, "bf16", parent, x, dt, A, Bm, Cm, D, h0)
    assert_parity(got, want, TOL["bf16"], f"rows kernel N={N} P={P} S={S} G={G}", kind="y")
    rounded = synth.round_to_bf16(h0)
    y = st.stree_tree_ssd(to_dev(parent), to_dev(x, "bf16"), to_dev(dt), to_dev(A), to_dev(Bm, "bf16"), to_dev(Cm, "bf16"),
                          to_dev(D), to_dev(rounded, "bf16"))
    same = _run_ssd(st, "bf16", parent, x, dt, A, Bm, Cm, D, rounded)
    assert np.array_equal(to_host(y), same)              # (a bf16 state is the operand that an fp32 one is rounded to)


@pytest.mark.parametrize("N", [100, 200])
def test_rows_kernel_large_values_and_positive_exponents(st, oracle, N):
    """exp(-s_j) alone is up to 2^64 where it is a factor of its own: inputs of 1e4 times the usual size stay finite, and
    steps that grow the state (A > 0) keep their weights."""
    B, H, P, S, G = 2, 3, 64, 128, 1
    parent = _trees(60 + N, B, N)
    x, dt, A, Bm, Cm, D, h0 = _rand(61 + N, "bf16", B, N, H, P, S, G)
    x = synth.round_to_bf16(x * 1e4)
    Bm, Cm = synth.round_to_bf16(Bm * 1e4), synth.round_to_bf16(Cm * 1e4)
    A[0], A[1], A[2] = -14.0, 0.5, -1.0
    want = oracle.ssd_paths(parent, x, dt, A, Bm, Cm, D, h0)
    got = _run_ssd(st, "bf16", parent, x, dt, A, Bm, Cm, D, h0)
    assert np.isfinite(got).all()
    assert_parity(got, want, TOL["bf16"], f"rows kernel, large values, N={N}", kind="y")


@pytest.mark.parametrize("N,Np", [(65, 1), (66, 64), (96, 65), (100, 17), (128, 128), (128, 256), (81, 200)])
@pytest.mark.parametrize("P,S,G,state", [(64, 128, 1, "f32"), (64, 64, 2, "bf16"), (64, 256, 1, "f32"), (128, 128, 2, "bf16"),
                                         (64, 64, 1, "f32"), (64, 128, 2, "bf16"), (64, 256, 1, "bf16"), (128, 128, 2, "f32")])
def test_replay_inside_the_rows_kernel(st, oracle, N, Np, P, S, G, state):
    """The state advanced inside the scan of a tree of 65 .. 128 nodes: accepted paths of one node, of more rows than are
    held at once (16), of more than a wave's lanes (64), none, and a previous tree that is refused."""
    import torch
    B, H = 7, 2
    parent, pparent = _trees(70 + N, B, N), _trees(71 + Np, B, Np)
    pparent[0] = pparent[1] = synth.chain_tree(Np)
    x, dt, A, Bm, Cm, D, h0 = _rand(72 + N, "bf16", B, N, H, P, S, G)
    px, pdt, _, pB, _, _, _ = _rand(73 + Np, "bf16", B, Np, H, P, S, G)
    if state == "bf16":
        h0 = synth.round_to_bf16(h0)
    acc = np.array([Np - 1, Np // 2, Np - 1, 0, -1, Np, Np // 3], dtype=np.int32)
    kept = np.where(acc >= Np, -1, acc).astype(np.int32)
    want_h, _ = oracle.commit(pparent, kept, px, pdt, A, pB, h0)
    h_in = to_dev(h0, "bf16") if state == "bf16" else to_dev(h0)
    status, rstatus = to_dev(np.full(B, 9, dtype=np.int32)), to_dev(np.full(B, 9, dtype=np.int32))
    args = (to_dev(pparent), to_dev(acc), to_dev(px, "bf16"), to_dev(pdt), to_dev(pB, "bf16"), to_dev(parent), to_dev(x, "bf16"),
            to_dev(dt), to_dev(A), to_dev(Bm, "bf16"), to_dev(Cm, "bf16"), to_dev(D))
    y, h = st.stree_tree_ssd_replay(*args, h_in, status=status, replay_status=rstatus)
    assert to_host(status).tolist() == [0] * B and to_host(rstatus).tolist() == [0, 0, 0, 0, 0, -1, 0]
    got_h = to_host(h)
    assert np.array_equal(got_h[4], h0[4]) and np.array_equal(got_h[5], h0[5])         # nothing accepted: passed through
    if state == "bf16":
        assert np.all(np.abs(got_h - want_h) <= 2.0 ** -8 * np.abs(want_h) + 1e-4 * np.abs(want_h).max())
        want_h = got_h.astype(np.float64)                                               # (the scan starts from what is written)
    else:
        assert_parity(got_h, want_h, 1e-4, f"replayed state N={N} Np={Np}", kind="state")
    want_y = oracle.ssd_paths(parent, x, dt, A, Bm, Cm, D, want_h)
    assert_parity(to_host(y), want_y, TOL["bf16"], f"scan behind the replay N={N} Np={Np}", kind="y")
    y2, _ = st.stree_tree_ssd_replay(*args, h_in, h_out=h_in)                           # in place
    assert torch.equal(y2, y) and torch.equal(h_in, h)


def test_replay_inside_the_rows_kernel_bad_trees(st, oracle):
    B, H, P, S, G, N, Np = 4, 2, 64, 128, 1, 90, 130
    parent, pparent = _trees(90, B, N), _trees(91, B, Np)
    parent[1, 70], pparent[2, 129] = 80, 129
    x, dt, A, Bm, Cm, D, h0 = _rand(92, "bf16", B, N, H, P, S, G)
    px, pdt, _, pB, _, _, _ = _rand(93, "bf16", B, Np, H, P, S, G)
    acc = np.full(B, Np // 2, dtype=np.int32)
    status, rstatus = to_dev(np.zeros(B, dtype=np.int32)), to_dev(np.zeros(B, dtype=np.int32))
    y, h = st.stree_tree_ssd_replay(to_dev(pparent), to_dev(acc), to_dev(px, "bf16"), to_dev(pdt), to_dev(pB, "bf16"),
                                    to_dev(parent), to_dev(x, "bf16"), to_dev(dt), to_dev(A), to_dev(Bm, "bf16"),
                                    to_dev(Cm, "bf16"), to_dev(D), to_dev(h0), status=status, replay_status=rstatus)
    assert to_host(status).tolist() == [0, 71, 0, 0] and to_host(rstatus).tolist() == [0, 0, 130, 0]
    ok = [0, 1, 3]
    want_h, _ = oracle.commit(pparent[ok], acc[ok], px[ok], pdt[ok], A, pB[ok], h0[ok])
    assert_parity(to_host(h)[ok], want_h, 1e-4, "state beside a bad tree", kind="state")
    assert np.array_equal(to_host(h)[2], h0[2]) and not np.any(to_host(y)[1])           # (the bad tree's state is replayed)
    for b, hb in ((0, want_h[0]), (2, h0[2].astype(np.float64)), (3, want_h[2])):
        want = oracle.ssd_paths(parent[b:b + 1], x[b:b + 1], dt[b:b + 1], A, Bm[b:b + 1], Cm[b:b + 1], D, hb[None])
        assert_parity(to_host(y)[b:b + 1], want, TOL["bf16"], f"scan beside a bad tree, sequence {b}", kind="y")
