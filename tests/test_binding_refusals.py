"""What the binding refuses before anything is launched, on the CPU: wrong shapes, types, strides and objects, entry point by
entry point, and that no argument of a call is lost on its way to the native half."""
import ctypes as C
import inspect
import os
import re

import numpy as np
import pytest
import torch

from paper_2505_14969_amd import binding as st

B, N, H, P, S, G, W, NP = 2, 6, 4, 64, 128, 2, 4, 5
CC = H * P + 2 * G * S
BF = torch.bfloat16


def _good():
    z = torch.zeros
    rows, prev = z(B, N, CC, dtype=BF), z(B, NP, CC, dtype=BF)
    x, Bm, Cm = z(B, N, H, P, dtype=BF), z(B, N, G, S, dtype=BF), z(B, N, G, S, dtype=BF)
    px, pB = z(B, NP, H, P, dtype=BF), z(B, NP, G, S, dtype=BF)
    par, ppar, acc = z(B, N, dtype=torch.int32), z(B, NP, dtype=torch.int32), z(B, dtype=torch.int32)
    dt, pdt, A, D, h0 = z(B, N, H), z(B, NP, H), z(H), z(H), z(B, H, P, S)
    cs, w, b = z(B, W - 1, CC, dtype=BF), z(CC, W, dtype=BF), z(CC, dtype=BF)
    heads = dict(nheads=H, headdim=P, dstate=S, ngroups=G)
    return {
        "stree_tree_conv": dict(parent=par, xbc_pre=rows, conv_state=cs, conv_w=w, conv_b=b, **heads),
        "stree_tree_ssd": dict(parent=par, x=x, dt=dt, A=A, Bm=Bm, Cm=Cm, D=D, h0=h0),
        "stree_commit_state": dict(parent=par, accepted=acc, x=x, dt=dt, A=A, Bm=Bm, h0=h0, xbc_pre=rows, conv_state=cs),
        "stree_tree_ssd_replay": dict(prev_parent=ppar, prev_accepted=acc, prev_x=px, prev_dt=pdt, prev_Bm=pB, parent=par, x=x,
                                      dt=dt, A=A, Bm=Bm, Cm=Cm, D=D, h0=h0),
        "stree_tree_conv_replay": dict(prev_parent=ppar, prev_accepted=acc, prev_xbc_pre=prev, parent=par, xbc_pre=rows,
                                       conv_state=cs, conv_w=w, conv_b=b, **heads),
        "stree_tree_step": dict(prev_parent=ppar, prev_accepted=acc, prev_xbc_pre=prev, prev_xbc_out=prev.clone(), prev_dt=pdt,
                                parent=par, xbc_pre=rows, conv_state=cs, conv_w=w, conv_b=b, dt=dt, A=A, D=D, h0=h0, **heads),
        "stree_gate_norm": dict(y=x, z=x.clone(), norm_w=torch.ones(H * P, dtype=BF), ngroups=G),
        "stree_linear_ssd": dict(x=x, dt=dt, A=A, Bm=Bm, Cm=Cm, D=D, h0=h0),
    }


def _strided(*shape, dtype=BF):                          # the right shape, rows twice as far apart
    return torch.zeros(*shape[:-1], 2 * shape[-1], dtype=dtype)[..., :shape[-1]]


REFUSED = [
    ("stree_tree_conv", "xbc_pre", lambda t: t[0], ValueError), ("stree_tree_conv", "xbc_pre", lambda t: t[..., :-8], AssertionError),
    ("stree_tree_conv", "xbc_pre", lambda t: t.double(), TypeError), ("stree_tree_conv", "nheads", lambda v: v + 1, AssertionError),
    ("stree_tree_conv", "nheads", lambda v: float(v), TypeError), ("stree_tree_conv", "conv_w", lambda t: _strided(CC, W), AssertionError),
    ("stree_tree_conv", "nheads", lambda v: v + 2 ** 32, AssertionError),                  # (not its low 32 bits)
    ("stree_tree_conv", "headdim", lambda v: v + 2 ** 64, AssertionError), ("stree_tree_conv_replay", "ngroups", lambda v: v - 2 ** 32, AssertionError),
    ("stree_tree_step", "dstate", lambda v: v + 2 ** 32, AssertionError),
    ("stree_tree_conv", "conv_state", lambda t: _strided(B, W - 1, CC), AssertionError),
    ("stree_tree_conv", "conv_state", lambda t: None, AttributeError),
    ("stree_tree_ssd", "x", lambda t: t[0], ValueError), ("stree_tree_ssd", "x", lambda t: t.double(), TypeError),
    ("stree_tree_ssd", "x", lambda t: t.float().numpy(), AttributeError), ("stree_tree_ssd", "Bm", lambda t: _strided(B, N, G, S), AssertionError),
    ("stree_tree_ssd", "Cm", lambda t: torch.zeros(B, 2 * N, G, S, dtype=BF)[:, :N], AssertionError),
    ("stree_tree_ssd", "dt", lambda t: t.double(), AssertionError), ("stree_tree_ssd", "dt", lambda t: _strided(B, N, H, dtype=torch.float32), AssertionError),
    ("stree_tree_ssd", "h0", lambda t: t.double(), TypeError), ("stree_tree_ssd", "out", lambda t: _strided(B, N, H, P), AssertionError),
    ("stree_tree_ssd", "dt_bias", lambda t: torch.zeros(H + 1), AssertionError), ("stree_tree_ssd", "dt_bias", lambda t: torch.zeros(H, dtype=BF), AssertionError),
    ("stree_tree_ssd", "parent", lambda t: [0], AttributeError),
    ("stree_commit_state", "x", lambda t: t[0], ValueError), ("stree_commit_state", "h_out", lambda t: torch.zeros(B, H, P, S, dtype=BF), AssertionError),
    ("stree_commit_state", "conv_state", lambda t: None, AttributeError), ("stree_commit_state", "accepted", lambda t: 0, AttributeError),
    ("stree_tree_ssd_replay", "prev_x", lambda t: t[:, :, :-1], AssertionError), ("stree_tree_ssd_replay", "prev_x", lambda t: t.float(), AssertionError),
    ("stree_tree_ssd_replay", "prev_dt", lambda t: t[:, :-1], AssertionError), ("stree_tree_ssd_replay", "prev_Bm", lambda t: t[:, :-1], AssertionError),
    ("stree_tree_ssd_replay", "h0", lambda t: _strided(B, H, P, S, dtype=torch.float32), AssertionError),
    ("stree_tree_ssd_replay", "h_out", lambda t: torch.zeros(B, H, P, S, dtype=BF), AssertionError),
    ("stree_tree_conv_replay", "prev_xbc_pre", lambda t: t[..., :-8], AssertionError),
    ("stree_tree_conv_replay", "conv_state_out", "conv_state", AssertionError),
    ("stree_tree_step", "prev_xbc_out", lambda t: t[:, :-1], AssertionError), ("stree_tree_step", "prev_dt", lambda t: t.double(), AssertionError),
    ("stree_tree_step", "dt", lambda t: _strided(B, N, H, dtype=torch.float32), AssertionError), ("stree_tree_step", "h0", lambda t: None, AttributeError),
    ("stree_tree_step", "conv_state_out", "conv_state", AssertionError), ("stree_tree_step", "dstate", lambda v: S // 2, AssertionError),
    ("stree_tree_step", "out", lambda t: _strided(B, N, H, P), AssertionError),
    ("stree_tree_step", "ngroups", lambda v: np.int64(v + 1), AssertionError),             # (numpy's integers are integers)
    ("stree_gate_norm", "z", lambda t: t.float(), AssertionError), ("stree_gate_norm", "z", lambda t: t[:, :-1], AssertionError),
    ("stree_gate_norm", "norm_w", lambda t: t[:-1], AssertionError), ("stree_gate_norm", "y", lambda t: _strided(B, N, H, P), AssertionError),
    ("stree_gate_norm", "y", lambda t: t[0], ValueError),
    ("stree_linear_ssd", "dt", lambda t: t[:, :-1], AssertionError), ("stree_linear_ssd", "h_out", lambda t: torch.zeros(B, H, P, S, dtype=BF), AssertionError),
    ("stree_linear_ssd", "x", lambda t: t.half(), TypeError), ("stree_linear_ssd", "Cm", lambda t: _strided(B, N, G, S), AssertionError),
]


@pytest.mark.parametrize("name,arg,change,error", REFUSED)
def test_refused_before_anything_is_launched(name, arg, change, error):
    call = _good()[name]
    call[arg] = call[change] if isinstance(change, str) else change(call.get(arg))
    with pytest.raises(error):
        getattr(st, name)(**call)


class _Like:
    """An array that is no tensor: the attributes of one that the binding asks for."""

    def __init__(self, t):
        self.t, self.shape, self.dtype = t, tuple(t.shape), t.dtype

    dim = lambda self: len(self.shape)
    stride = lambda self: self.t.stride()
    is_contiguous = lambda self: self.t.is_contiguous()
    numel = lambda self: self.t.numel()
    element_size = lambda self: self.t.element_size()
    data_ptr = lambda self: self.t.data_ptr()


class _Own(torch.Tensor):
    """A tensor whose address and density are its own methods'."""
    asked = []

    def data_ptr(self):
        self.asked.append("data_ptr")
        return super().data_ptr()

    def is_contiguous(self):
        return True


@pytest.fixture
def nothing_launched():
    """The entry points replaced by one that returns at once, so that no call goes further than that on any machine."""
    entry = C.CFUNCTYPE(C.c_int, C.c_void_p)(lambda dims: 0)
    st._native().bind(st.StreeError, *[C.cast(entry, C.c_void_p).value] * len(st._ENTRIES))
    yield
    st._bind(st.load())


def _outcome(name, call):
    try:
        getattr(st, name)(**call)
    except RuntimeError as e:                            # no GPU here: the checks are passed, the stream is asked for
        return str(e).splitlines()[0]
    return "launched"


# (the rows themselves, whose type decides the kernels, are tensors)
ROWS = {"stree_tree_conv": "xbc_pre", "stree_tree_ssd": "x", "stree_commit_state": "x", "stree_tree_ssd_replay": "x",
        "stree_tree_conv_replay": "xbc_pre", "stree_tree_step": "xbc_pre", "stree_gate_norm": "y", "stree_linear_ssd": "x"}


@pytest.mark.parametrize("name", sorted(ROWS))
def test_arrays_that_are_no_tensors_are_taken(name, nothing_launched):
    call = _good()[name]
    want = _outcome(name, call)
    for arg, value in call.items():
        if not isinstance(value, torch.Tensor):
            continue
        changed = dict(call)
        if arg != ROWS[name]:
            changed[arg] = _Like(value)
            result = {"h0": "h_out", "conv_state": "conv_state_out"}.get(arg)
            if result in inspect.signature(getattr(st, name)).parameters:        # (nothing can be made like them)
                changed[result] = torch.empty_like(value)
            assert _outcome(name, changed) == want, arg
        changed[arg] = value.as_subclass(_Own)
        _Own.asked.clear()
        assert _outcome(name, changed) == want and "data_ptr" in _Own.asked, arg


def test_a_torch_function_mode_sees_the_calls(nothing_launched):
    from torch.overrides import TorchFunctionMode
    seen = set()

    class Listener(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.add(getattr(func, "__name__", str(func)))
            return func(*args, **(kwargs or {}))
    call = _good()["stree_gate_norm"]
    with Listener():
        _outcome("stree_gate_norm", call)
    assert {"data_ptr", "empty_like", "is_contiguous"} <= seen


# host.cpp's short names of arguments
SHORT = {"pparent": "prev_parent", "paccepted": "prev_accepted", "px": "prev_x", "pdt": "prev_dt", "pBm": "prev_Bm",
         "pxbc_pre": "prev_xbc_pre", "pxbc_out": "prev_xbc_out", "rstatus": "replay_status"}


def _native_order():
    """Per entry point the arguments in the order in which host.cpp numbers them, and how many it says it takes."""
    with open(os.path.join(os.path.dirname(os.path.abspath(st.__file__)), "csrc", "host.cpp")) as f:
        text = f.read()
    order = {}
    for name, function, count in re.findall(r'STREE_METHOD\("(\w+)", (\w+), (\d+)\)', text):
        body = re.search(r"PyObject \*%s\(const Args &a\) \{\s*enum \{([^}]*)\}" % function, text).group(1)
        order["stree_" + name] = ([SHORT.get(n, n) for n in re.findall(r"\w+", body)], int(count))
    return order


def test_every_argument_reaches_the_native_half():
    """The functions pass their arguments by position: each at the place, and as many, as the other side reads."""
    class Seen:
        def __getattr__(self, entry):
            return lambda *args: args
    order = _native_order()
    assert sorted(order) == sorted(_good())
    kept, st._host = st._native(), Seen()
    try:
        for name, (names, count) in order.items():
            f = getattr(st, name)
            passed = f(**{n: n for n in inspect.signature(f).parameters})
            assert list(passed) == names and len(passed) == count, name
    finally:
        st._host = kept
