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
