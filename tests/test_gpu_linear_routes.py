"""The prefix scan on each of its routes, at the sizes where they begin, end and leave remainders, against the
oracle's causal scan (bounds as in test_gpu_linear.py: state 1e-4, y one bf16 product chain)."""
import numpy as np
import pytest

from paper_2505_14969_amd import synth
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


@pytest.mark.parametrize("B,T,H,P,S,G", ROUTES)
def test_prefix_routes_with_a_bf16_state(st, oracle, B, T, H, P, S, G):
    """The state's way between memory and the accumulators in both types: in place, and from an fp32 state of the same
    values (which both forms widen exactly: y equal, the bf16 state the rounded fp32 one)."""
    import torch
    x, dt, A, Bm, Cm, D, h0 = _rand(1900 + T, "bf16", B, T, H, P, S, G, h0=True)
    h0 = synth.round_to_bf16(h0)
    want_y, want_h = oracle.linear_scan(x, dt, A, Bm, Cm, D, h0)
    args = (to_dev(x, "bf16"), to_dev(dt), to_dev(A), to_dev(Bm, "bf16"))
    y32, h32 = st.stree_linear_ssd(*args, to_dev(Cm, "bf16"), to_dev(D), to_dev(h0))
    h = to_dev(h0, "bf16")
    y, _ = st.stree_linear_ssd(*args, to_dev(Cm, "bf16"), to_dev(D), h, h_out=h)
    assert_parity(to_host(y), want_y, TOL["bf16"], f"y of {T} tokens", kind="y")
    assert torch.equal(y, y32) and torch.equal(h, h32.bfloat16())
    h2 = to_dev(h0, "bf16")
    st.stree_linear_ssd(*args, h0=h2, want_y=False, h_out=h2)
    for got in (to_host(h), to_host(h2)):              # one rounding (2^-8 relative) of a state within 1e-4
        assert np.all(np.abs(got - want_h) <= 2.0 ** -8 * np.abs(want_h) + 1e-4 * np.abs(want_h).max())


# the routes that walk a sequence in segments: with y from 705 tokens on, state only from 449 on, four segments there
# once eight waves a column group are more than the chip holds at two a SIMD
SEGMENTS = [(1, 449, 3, 64, 128, 1), (1, 450, 132, 64, 128, 2), (2, 705, 4, 64, 64, 2), (1, 1013, 2, 64, 128, 1),
            (2, 705, 2, 128, 128, 2), (1, 460, 260, 64, 64, 1), (1, 1013, 2, 64, 256, 1)]


@pytest.mark.parametrize("state", ["f32", "bf16"])
@pytest.mark.parametrize("B,T,H,P,S,G", SEGMENTS)
def test_prefix_segments_with_every_option(st, oracle, B, T, H, P, S, G, state):
    """No initial state, no D, raw step sizes with a bias, and a head whose decay underflows within a few tokens (the
    chain's factor exp(sum s) is then 0 for every segment)."""
    import torch
    x, _, A, Bm, Cm, D, h0 = _rand(2900 + T + H, "bf16", B, T, H, P, S, G, h0=True)
    h0 = synth.round_to_bf16(h0) if state == "bf16" else h0
    rng = np.random.default_rng(T)
    raw, bias = rng.standard_normal((B, T, H)).astype(np.float32), rng.uniform(-3.0, -1.0, H).astype(np.float32)
    A[H - 1], bias[H - 1] = -100.0, 0.5
    dt = oracle.step_size(raw, bias)
    dx, dB, dC = to_dev(x, "bf16"), to_dev(Bm, "bf16"), to_dev(Cm, "bf16")
    for with_h0, with_D in ((True, False), (False, True)):
        opt = (D if with_D else None, h0 if with_h0 else None)
        want_y, want_h = oracle.linear_scan(x, dt, A, Bm, Cm, *opt)
        # y: the weights M or the state, and the result, are rounded to bf16 (2^-9 relative each) in front of sums of
        # terms that are no larger than those of the scan of absolute values
        terms, _ = oracle.linear_scan(abs(x), dt, A, abs(Bm), abs(Cm), *[None if a is None else abs(a) for a in opt])
        for want in (True, False):
            h = torch.empty((B, H, P, S), dtype=torch.bfloat16 if state == "bf16" else torch.float32, device="cuda")
            y, _ = st.stree_linear_ssd(dx, to_dev(raw), to_dev(A), dB, dC if want else None,
                                       to_dev(D) if with_D and want else None, to_dev(h0, state) if with_h0 else None,
                                       want_y=want, h_out=h, dt_bias=to_dev(bias))
            what = f"h0 {with_h0}, D {with_D}, y {want}"
            if want:
                err = np.abs(to_host(y) - want_y)
                assert np.all(err <= 2.0 ** -8 * terms) and np.linalg.norm(err) <= TOL["bf16"] * np.linalg.norm(want_y), what
            got = to_host(h)
            assert np.isfinite(got).all()
            for k in range(H):                         # head by head: the underflowing one has a scale of its own
                bound = 1e-4 * np.abs(want_h[:, k]).max() + (2.0 ** -8 * np.abs(want_h[:, k]) if state == "bf16" else 0.0)
                assert np.all(np.abs(got[:, k] - want_h[:, k]) <= bound), f"state of head {k}, {what}"


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


def test_prefix_of_more_heads_than_one_grid_dimension_holds(st):
    """257 x 65535 heads of one token (a state of 138 GB in bf16): as one workgroup each, more than 2^32 work items; whole
    sequences go as several launches.  Closed forms at one token: h = dt x (outer) B, y = (dt <B, C> + D) x."""
    import torch
    B, T, H, P, S, G = 257, 1, 65535, 64, 64, 1
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 160 << 30:
        pytest.skip("needs 160 GB of free device memory")
    gen = torch.Generator(device="cuda").manual_seed(4)
    rand = lambda *s: torch.randn(s, generator=gen, device="cuda").to(torch.bfloat16)  # noqa: E731
    x, Bm, Cm = rand(B, T, H, P), rand(B, T, G, S), rand(B, T, G, S)
    dt = torch.rand((B, T, H), generator=gen, device="cuda")
    A, D = -torch.rand(H, generator=gen, device="cuda"), torch.randn(H, generator=gen, device="cuda")
    h = torch.full((B, H, P, S), 7.0, dtype=torch.bfloat16, device="cuda")
    y = st.stree_linear_ssd(x, dt, A, Bm, Cm, D, h_out=h)[0]
    wrong = []
    for b in (0, 14, 15, 16, 17, 128, 255, 256):       # (16 sequences a launch)
        w = dt[b, 0, :, None] * x[b, 0].float()
        want_h = w[:, :, None] * Bm[b, 0, 0].float()
        bc = (Bm[b, 0, 0].float() * Cm[b, 0, 0].float()).sum()
        want = w * bc + D[:, None] * x[b, 0].float()
        ok_h = ((h[b].float() - want_h).abs() <= 2.0 ** -8 * want_h.abs() + 1e-4).all()
        # M = dt <B, C> and the result are rounded to bf16
        ok_y = ((y[b, 0].float() - want).abs() <= 2.0 ** -8 * (want.abs() + 1.1 * (w * bc).abs()) + 1e-6).all()
        wrong += [] if bool(ok_h) and bool(ok_y) else [b]
    del h, want_h
    torch.cuda.empty_cache()
    assert not wrong
