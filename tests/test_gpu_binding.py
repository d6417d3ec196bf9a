"""The binding on the GPU with arrays that are not plain tensors: the same step, bit for bit."""
import numpy as np
import pytest

from paper_2505_14969_amd import synth
from helpers import to_dev
from test_binding_refusals import _Like, _Own
from test_gpu_parity import _trees, st  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def test_step_with_arrays_of_every_kind(st):
    import torch
    B, N, Np, H, P, S, G, W = 2, 9, 5, 4, 64, 128, 2, 4
    Cc, gen = H * P + 2 * G * S, torch.Generator(device="cuda").manual_seed(3)

    def rand(*shape, dtype=torch.bfloat16):
        return torch.randn(shape, generator=gen, device="cuda").to(dtype)
    f32 = torch.float32
    args = dict(prev_parent=to_dev(_trees(1, B, Np)), prev_accepted=to_dev(np.array([4, 2], dtype=np.int32)),
                prev_xbc_pre=rand(B, Np, Cc), prev_xbc_out=rand(B, Np, Cc), prev_dt=rand(B, Np, H, dtype=f32).abs(),
                parent=to_dev(np.stack([synth.chain_tree(N)] * B)), xbc_pre=rand(B, N, Cc), conv_state=rand(B, W - 1, Cc),
                conv_w=rand(Cc, W), conv_b=rand(Cc), dt=rand(B, N, H, dtype=f32).abs(), A=-rand(H, dtype=f32).abs(),
                D=rand(H, dtype=f32), h0=rand(B, H, P, S, dtype=f32), nheads=H, headdim=P, dstate=S, ngroups=G)
    want = st.stree_tree_step(**args)
    results = dict(h_out=torch.empty_like(args["h0"]), conv_state_out=torch.empty_like(args["conv_state"]))
    alike = {k: _Like(v) if isinstance(v, torch.Tensor) and k != "xbc_pre" else v for k, v in args.items()}
    own = {k: v.as_subclass(_Own) if isinstance(v, torch.Tensor) else v for k, v in args.items()}
    held = {k: torch.nn.Parameter(v, requires_grad=False) if k in ("A", "D", "conv_w", "conv_b") else v for k, v in args.items()}
    for got in (st.stree_tree_step(**alike, **results), st.stree_tree_step(**own), st.stree_tree_step(**held)):
        for a, b in zip(got, want):
            assert torch.equal(a.as_subclass(torch.Tensor), b)
