"""GPU parity of the commit on trees of more than 64 nodes, whose path is found in groups of 64 nodes: paths that stay in
one group, cross several, end at a group's first or last node, and groups that are filled in part."""
import numpy as np
import pytest

from paper_2505_14969_amd import synth
from helpers import assert_parity, to_dev, to_host
from test_gpu_parity import _rand, _trees, st  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("N", [65, 127, 128, 129, 192, 193, 256])
def test_commit_path_across_groups(st, oracle, N, io):
    ends = sorted({0, 63, 64, N // 2, N - 1, min(128, N - 1), min(191, N - 1)})
    B, H, P, S, G = 2 * len(ends) + 2, 2, 64, 128, 1
    acc = np.array(ends + ends + [-1, N], dtype=np.int32)             # (-1: nothing accepted; N: refused, state kept)
    parent = _trees(700 + N, B, N)
    parent[:len(ends)] = synth.chain_tree(N)                          # the longest paths: every group, every node
    parent[len(ends), 1:] = np.where(np.arange(1, N) < 64, 0, np.arange(1, N) - 64)   # a path of one node a group
    x, dt, A, Bm, _, _, h0 = _rand(701 + N, io, B, N, H, P, S, G)
    want, _ = oracle.commit(parent[:-1], acc[:-1], x[:-1], dt[:-1], A, Bm[:-1], h0[:-1])
    status = to_dev(np.full(B, 9, dtype=np.int32))
    h, _ = st.stree_commit_state(to_dev(parent), to_dev(acc), to_dev(x, io), to_dev(dt), to_dev(A), to_dev(Bm, io),
                                 to_dev(h0), status=status)
    got = to_host(h)
    for b in range(B - 1):
        assert_parity(got[b], want[b], 1e-4, f"commit, N={N}, {io}, accepted {acc[b]}, sequence {b}", kind="state")
    assert np.array_equal(got[-1], h0[-1])
    assert to_host(status).tolist() == [0] * (B - 1) + [-1]


def test_commit_bad_tree_in_any_group(st):
    B, N, H, P, S, G = 4, 200, 2, 64, 128, 1
    parent = _trees(800, B, N)
    parent[1, 70], parent[1, 180] = 70, 199                           # the first bad node of several is reported
    parent[2, 199] = -1
    x, dt, A, Bm, _, _, h0 = _rand(801, "bf16", B, N, H, P, S, G)
    status = to_dev(np.full(B, 9, dtype=np.int32))
    h, _ = st.stree_commit_state(to_dev(parent), to_dev(np.full(B, N - 1, dtype=np.int32)), to_dev(x, "bf16"), to_dev(dt),
                                 to_dev(A), to_dev(Bm, "bf16"), to_dev(h0), status=status)
    assert to_host(status).tolist() == [0, 71, 200, 0]
    got = to_host(h)
    assert np.array_equal(got[1], h0[1]) and np.array_equal(got[2], h0[2]) and not np.array_equal(got[0], h0[0])
