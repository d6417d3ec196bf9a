"""The prefix scan where the heads left over from 256 or 512 are worked on as two halves of 32 columns, at the lines of
that rule (256 and 512: none are left over; 384 the most that are split, 385 one more; 641 more halves than the chip
holds at once), against the oracle's causal scan (bounds as in test_gpu_linear.py: state 1e-4, y one bf16 product chain)."""
import pytest

from paper_2505_14969_amd import synth
from helpers import TOL, assert_parity, to_dev, to_host
from test_gpu_parity import _rand, st  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

# (B, T, H, S, G)
LINES = [(1, 33, 256, 128, 1), (1, 65, 257, 128, 1), (3, 31, 91, 128, 1), (2, 97, 192, 64, 2), (5, 32, 77, 128, 7),
         (1, 64, 384, 256, 4), (1, 40, 513, 256, 1), (4, 70, 130, 128, 2), (2, 1, 320, 128, 1), (1, 34, 641, 64, 1)]


@pytest.mark.parametrize("state", ["f32", "bf16"])
@pytest.mark.parametrize("B,T,H,S,G", LINES)
def test_prefix_of_heads_left_over(st, oracle, B, T, H, S, G, state):
    x, dt, A, Bm, Cm, D, h0 = _rand(4900 + T + H, "bf16", B, T, H, 64, S, G, h0=True)
    h0 = synth.round_to_bf16(h0) if state == "bf16" else h0
    args = (to_dev(x, "bf16"), to_dev(dt), to_dev(A), to_dev(Bm, "bf16"), to_dev(Cm, "bf16"))
    # a bf16 state (8 significant bits) is rounded once more when it is stored: by 2^-8 of its value at most
    tol = 1e-4 + (2.0 ** -8 if state == "bf16" else 0.0)
    want_y, want_h = oracle.linear_scan(x, dt, A, Bm, Cm, D, h0)
    h = to_dev(h0, state) if state == "bf16" else to_dev(h0)
    y, _ = st.stree_linear_ssd(*args, to_dev(D), h, h_out=h)          # in place: each half owns its rows of the state
    assert_parity(to_host(y), want_y, TOL["bf16"], f"y of {B * H} heads", kind="y")
    assert_parity(to_host(h), want_h, tol, f"state of {B * H} heads", kind="state")
    want_y, want_h = oracle.linear_scan(x, dt, A, Bm, Cm, None, None)
    y, h = st.stree_linear_ssd(*args)
    assert_parity(to_host(y), want_y, TOL["bf16"], f"y of {B * H} heads from zero", kind="y")
    assert_parity(to_host(h), want_h, 1e-4, f"state of {B * H} heads from zero", kind="state")
