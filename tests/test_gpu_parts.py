"""GPU parity of the tree kernels with more heads than one launch takes (2^21): the sequences of the second and third
launch have their own trees, rows, states and status words."""
import numpy as np
import pytest

from paper_2505_14969_amd import synth
from helpers import TOL, assert_parity, to_dev, to_host
from test_gpu_parity import _trees, st  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

H = 65535                                                # 32 sequences a launch
SLICES = (slice(0, 3), slice(H - 3, H))


def _inputs(seed, B, N, S, groups=1):
    """x, dt, A, B, C, D, made on the GPU.  Without D where there are few rows: dt <C, B> + D may cancel, and nothing else
    sets the scale that errors are measured by."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.empty((B, N, H, 64), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    rows = [torch.randn((B, N, groups, S), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2)]
    dt = torch.rand((B, N, H), generator=gen, device="cuda") * 0.2
    A, D = -torch.exp(torch.rand(H, generator=gen, device="cuda") * 2), torch.randn(H, generator=gen, device="cuda")
    return x, dt, A, rows[0], rows[1], D if N > 3 else None


def _check_y(oracle, y, parent, ins, h0, b, what):
    x, dt, A, Bm, Cm, D = ins
    for s in SLICES:
        state = None if h0 is None else to_host(h0[b:b + 1, s])
        want = oracle.ssd_paths(parent[b:b + 1], to_host(x[b:b + 1, :, s]), to_host(dt[b:b + 1, :, s]), to_host(A[s]),
                                to_host(Bm[b:b + 1]), to_host(Cm[b:b + 1]), None if D is None else to_host(D[s]), state)
        assert_parity(to_host(y[b:b + 1, :, s]), want, TOL["bf16"], f"{what}, sequence {b}, heads from {s.start}", kind="y")


@pytest.mark.parametrize("B,N", [(65, 2), (33, 65)])
def test_scan_in_several_launches(st, oracle, B, N):
    parent, ins = _trees(900 + N, B, N), _inputs(901 + N, B, N, 64)
    refused = parent.copy()
    refused[B - 1, 1] = 1                                # the last sequence's tree
    for tree, last in ((refused, 2), (parent, 0)):
        status = to_dev(np.full(B, 9, dtype=np.int32))
        y = st.stree_tree_ssd(to_dev(tree), *ins, status=status)
        assert to_host(status).tolist() == [0] * (B - 1) + [last]
        for b in sorted({0, 31, 32, B - 2, B - 1}):
            if b == B - 1 and last:
                assert not y[b].any()
            else:
                _check_y(oracle, y, tree, ins, None, b, f"scan of {B} x {N} nodes")


@pytest.mark.parametrize("B,N,Np", [(65, 2, 3), (33, 65, 3)])
def test_replay_in_several_launches(st, oracle, B, N, Np):
    import torch
    S = 64
    parent, pparent = _trees(910 + N, B, N), _trees(911, B, Np)
    ins, prev = _inputs(912 + N, B, N, S), _inputs(913 + N, B, Np, S)
    h = torch.empty((B, H, 64, S), dtype=torch.bfloat16, device="cuda").normal_(std=0.1)
    acc = (np.arange(B) % Np).astype(np.int32)
    acc[B - 1] = Np                                      # refused: the last sequence's state passes through
    seen = sorted({0, 31, 32, B - 2, B - 1})
    before = {b: [to_host(h[b:b + 1, s]) for s in SLICES] for b in seen}
    status, rstatus = to_dev(np.full(B, 9, dtype=np.int32)), to_dev(np.full(B, 9, dtype=np.int32))
    px, pdt, _, pB, _, _ = prev
    x, dt, A, Bm, Cm, D = ins
    y, h = st.stree_tree_ssd_replay(to_dev(pparent), to_dev(acc), px, pdt, pB, to_dev(parent), x, dt, A, Bm, Cm, D, h,
                                    h_out=h, status=status, replay_status=rstatus)
    assert to_host(status).tolist() == [0] * B and to_host(rstatus).tolist() == [0] * (B - 1) + [-1]
    for b in seen:
        for was, s in zip(before[b], SLICES):
            got = to_host(h[b:b + 1, s])
            if b == B - 1:
                assert np.array_equal(got, was)
                continue
            want, _ = oracle.commit(pparent[b:b + 1], acc[b:b + 1], to_host(px[b:b + 1, :, s]), to_host(pdt[b:b + 1, :, s]),
                                    to_host(A[s]), to_host(pB[b:b + 1]), was)
            # a bf16 state (8 significant bits) is rounded once more when it is stored: by 2^-8 of its value at most
            assert np.all(np.abs(got - want) <= 2.0 ** -8 * np.abs(want) + 1e-4 * np.abs(want).max()), f"state {b}"
        _check_y(oracle, y, parent, ins, h, b, f"replay, {B} x {N} nodes")
