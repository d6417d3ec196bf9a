"""The prefix scan on each of its routes, at the sizes where they begin, end and leave remainders, against the
oracle's causal scan (bounds as in test_gpu_linear.py: state 1e-4, y one bf16 product chain)."""
import numpy as np
import pytest

from helpers import TOL, assert_parity, to_dev, to_host
from test_gpu_parity import _rand, st  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

# (B, T, H, P, S, G): with y, segments of one sequence from 705 tokens on while the chip is not full, teams else;
# state only, segments from 449 tokens on (four of them from 129 / 257 heads on)
ROUTES = [(1, 31, 3, 64, 128, 1), (1, 33, 2, 64, 64, 1), (2, 95, 2, 64, 256, 2), (1, 97, 2, 128, 128, 1),   # teams
          (1, 448, 2, 64, 128, 1), (2, 449, 4, 64, 128, 2), (1, 513, 2, 64, 64, 1), (1, 450, 2, 64, 256, 1),
          (1, 704, 2, 128, 128, 2), (1, 705, 2, 64, 128, 1), (2, 1013, 2, 64, 64, 2), (1, 769, 2, 128, 128, 1),
          (1, 450, 132, 64, 128, 1), (1, 460, 260, 64, 64, 2), (1, 720, 132, 64, 128, 4)]


@pytest.mark.parametrize("B,T,H,P,S,G", ROUTES)
def test_prefix_routes(st, oracle, B, T, H, P, S, G):
    x, dt, A, Bm, Cm, D, h0 = _rand(900 + T, "bf16", B, T, H, P, S, G, h0=True)
    want_y, want_h = oracle.linear_scan(x, dt, A, Bm, Cm, D, h0)
    args = (to_dev(x, "bf16"), to_dev(dt), to_dev(A), to_dev(Bm, "bf16"))
    h = to_dev(h0)                                    # in place: h0 is still read when the last segment's state is there
    y, _ = st.stree_linear_ssd(*args, to_dev(Cm, "bf16"), to_dev(D), h, h_out=h)
    assert_parity(to_host(h), want_h, 1e-4, f"state after {T} tokens", kind="state")
    assert_parity(to_host(y), want_y, TOL["bf16"], f"y of {T} tokens", kind="y")
    h = to_dev(h0)
    st.stree_linear_ssd(*args, h0=h, want_y=False, h_out=h)
    assert_parity(to_host(h), want_h, 1e-4, f"state only after {T} tokens", kind="state")


def test_prefix_with_huge_token_strides(st, oracle):
    """Rows 64 MiB apart: beyond the 32-bit offsets of the ordinary form (17 GB, of which three columns are used; up
    to 256 tokens the entry point refuses such strides)."""
    import torch
    B, T, H, P, S, G, stride = 1, 257, 2, 64, 128, 1, 1 << 25
    x, dt, A, Bm, Cm, D, h0 = _rand(5, "bf16", B, T, H, P, S, G, h0=True)
    want_y, want_h = oracle.linear_scan(x, dt, A, Bm, Cm, D, h0)
    room = torch.empty(T * stride, dtype=torch.bfloat16, device="cuda").view(1, T, stride)
    views = []
    for k, (a, n) in enumerate(((x, H * P), (Bm, G * S), (Cm, G * S))):
        v = room[:, :, 1024 * k:1024 * k + n]
        v.copy_(to_dev(a, "bf16").reshape(1, T, n))
        views.append(v.unflatten(2, a.shape[2:]))
    y, h = st.stree_linear_ssd(views[0], to_dev(dt), to_dev(A), views[1], views[2], to_dev(D), to_dev(h0))
    assert_parity(to_host(h), want_h, 1e-4, "state", kind="state")
    assert_parity(to_host(y), want_y, TOL["bf16"], "y", kind="y")
    _, h2 = st.stree_linear_ssd(views[0], to_dev(dt), to_dev(A), views[1], h0=to_dev(h0), want_y=False)
    assert_parity(to_host(h2), want_h, 1e-4, "state only", kind="state")


@pytest.mark.parametrize("P,S", [(64, 64), (64, 128), (64, 256), (128, 128)])
@pytest.mark.parametrize("T", [1, 31, 33, 65, 449, 705])
def test_prefix_reads_nothing_behind_the_last_token(st, oracle, T, P, S):
    """x, B and C are the first T rows of a longer buffer whose other rows are NaN (a weight of 0 would not hide one)."""
    import torch
    B, H, G = 1, 2, 1
    x, dt, A, Bm, Cm, D, h0 = _rand(1300 + T + S, "bf16", B, T, H, P, S, G, h0=True)
    want_y, want_h = oracle.linear_scan(x, dt, A, Bm, Cm, D, h0)
    views = []
    for a, n in ((x, H * P), (Bm, G * S), (Cm, G * S)):
        rows = torch.full((B, T + 192, n), float("nan"), dtype=torch.bfloat16, device="cuda")
        rows[:, :T] = to_dev(a, "bf16").reshape(B, T, n)
        views.append(rows[:, :T].unflatten(2, a.shape[2:]))
    y, h = st.stree_linear_ssd(views[0], to_dev(dt), to_dev(A), views[1], views[2], to_dev(D), to_dev(h0))
    assert_parity(to_host(h), want_h, 1e-4, "state", kind="state")
    assert_parity(to_host(y), want_y, TOL["bf16"], "y", kind="y")
    _, h2 = st.stree_linear_ssd(views[0], to_dev(dt), to_dev(A), views[1], h0=to_dev(h0), want_y=False)
    assert_parity(to_host(h2), want_h, 1e-4, "state only", kind="state")
