"""The prefix scan without y at the lines of its dispatch -- one, two and four segments of a sequence, 32 and 64
columns a wave, by the column groups (of 32) and the pairs of 32-token chunks -- against the oracle's causal scan (bound of
the state as in test_gpu_linear.py: 1e-4)."""
import pytest

from paper_2505_14969_amd import synth
from helpers import assert_parity, to_dev, to_host
from test_gpu_parity import _rand, st  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

# (B, T, H, P, S, G)
LINES = [(1, 1, 3, 64, 128, 1), (2, 65, 3, 128, 128, 1), (1, 448, 4, 64, 128, 2), (1, 66, 255, 64, 64, 1),     # below 8 pairs
         (1, 66, 256, 64, 64, 1), (4, 130, 128, 64, 128, 1), (4, 60, 64, 64, 128, 1), (1, 193, 2, 64, 256, 2),
         (1, 449, 4, 64, 128, 2), (1, 700, 128, 64, 64, 1), (1, 1013, 64, 64, 256, 2), (2, 512, 3, 128, 128, 1),  # few groups
         (1, 449, 129, 64, 128, 3), (2, 576, 128, 64, 64, 1), (1, 550, 65, 64, 256, 1),                        # 8 and 9 pairs
         (4, 576, 128, 64, 64, 2), (4, 449, 128, 64, 128, 1),
         (1, 577, 129, 64, 128, 1), (2, 640, 65, 64, 64, 1), (1, 609, 65, 128, 128, 1), (1, 1025, 65, 64, 256, 1),
         (1, 1729, 3, 64, 256, 1), (1, 1728, 3, 64, 256, 1), (2, 449, 65, 64, 64, 5), (2, 641, 72, 64, 128, 1),  # both sides of each line
         (2, 640, 72, 64, 128, 1), (1, 1217, 129, 64, 128, 3), (2, 1473, 33, 64, 256, 1), (2, 1472, 33, 64, 256, 1),
         (2, 640, 130, 64, 128, 2), (2, 705, 130, 64, 128, 1), (2, 1217, 152, 64, 64, 1), (2, 1216, 152, 64, 64, 1),
         (1, 3009, 152, 64, 256, 1), (3, 641, 128, 64, 128, 1), (3, 577, 128, 64, 64, 1), (4, 1217, 130, 64, 128, 1),
         (4, 1216, 65, 128, 128, 1), (5, 449, 26, 64, 256, 1), (8, 705, 82, 64, 128, 1), (8, 641, 112, 64, 128, 1)]


@pytest.mark.parametrize("state", ["f32", "bf16"])
@pytest.mark.parametrize("B,T,H,P,S,G", LINES)
def test_state_only(st, oracle, B, T, H, P, S, G, state):
    x, dt, A, Bm, Cm, D, h0 = _rand(5900 + T + H, "bf16", B, T, H, P, S, G, h0=True)
    h0 = synth.round_to_bf16(h0) if state == "bf16" else h0
    args = (to_dev(x, "bf16"), to_dev(dt), to_dev(A), to_dev(Bm, "bf16"))
    # a bf16 state (8 significant bits) is rounded once more when it is stored: by 2^-8 of its value at most
    tol = 1e-4 + (2.0 ** -8 if state == "bf16" else 0.0)
    _, want = oracle.linear_scan(x, dt, A, Bm, Cm, None, h0)
    h = to_dev(h0, "bf16") if state == "bf16" else to_dev(h0)
    st.stree_linear_ssd(*args, h0=h, want_y=False, h_out=h)           # in place
    assert_parity(to_host(h), want, tol, f"state after {T} tokens", kind="state")
    _, want = oracle.linear_scan(x, dt, A, Bm, Cm, None, None)
    _, h = st.stree_linear_ssd(*args, want_y=False)
    assert_parity(to_host(h), want, 1e-4, f"state after {T} tokens from zero", kind="state")


@pytest.mark.parametrize("B,T,H,P,S", [(1, 512, 4, 64, 64), (1, 512, 129, 64, 64), (1, 640, 260, 64, 128)])
def test_state_of_zeros_behind_steps_that_grow(st, oracle, B, T, H, P, S):
    """Steps with A > 0 whose growth over all later segments is beyond fp32's range, from a state of zeros: nothing grows
    until x comes, in the last segment."""
    x, dt, A, Bm, _, _, _ = _rand(6400 + H, "bf16", B, T, H, P, S, 1)
    x[:, :T - 128] = 0.0
    dt[:] = 0.5
    A[:] = 0.55                                          # 0.4 bits a token: 2^51 a segment of 128, 2^152 for three
    _, want = oracle.linear_scan(x, dt, A, Bm, Bm, None, None)
    _, h = st.stree_linear_ssd(to_dev(x, "bf16"), to_dev(dt), to_dev(A), to_dev(Bm, "bf16"), want_y=False)
    assert_parity(to_host(h), want, 1e-4, f"state behind {T - 128} empty tokens", kind="state")
