"""The work that a user of this library has it do, as cases that can be timed and compared.

A case is one layer's pass of one of three kinds, through the binding's public calls:

  step     a decoding iteration as the README shows it: ``stree_tree_step`` (tree conv, replay of the previous
           tree's accepted path, tree scan) and ``stree_gate_norm`` behind it
  verify   the same iteration with the commit done at its end: ``stree_tree_conv``, ``stree_tree_ssd``, the gate and
           norm, ``stree_commit_state`` (with ``conv`` False the activations come from elsewhere: scan and commit)
  prefill  ``stree_linear_ssd`` over a prompt: outputs and state, or (``want_y`` False) the state only

Layer shapes are the repository's configurations (80 heads x 64 with dstate 128, 128 heads in 8 groups, the 4-head fp32
layer) and the other head shapes that its tests run (dstate 64 and 256, headdim 128).  Trees are the paper's: full
binary trees of 15 / 31 / 63 tokens, beams of M tokens a layer (29 to 81 nodes), random trees of depth 4 to 10, chains.
Values follow the recipe of ``synth.draw_tensors``; activations behind the conv have a SiLU's distribution.
"""
import math

import numpy as np
import torch

from paper_2505_14969_amd import binding as st
from paper_2505_14969_amd import synth

CONV_WIDTH = 4


def _case(kind, batch, heads=80, headdim=64, dstate=128, groups=1, dtype="bf16", state="f32", softplus=False, **more):
    return dict(kind=kind, batch=batch, heads=heads, headdim=headdim, dstate=dstate, groups=groups, dtype=dtype,
                state=state, softplus=softplus, **more)


def listed():
    cases = [
        # one user, a small static or binary draft tree: launches and host time count as much as the kernels
        _case("step", 1, nodes=15, prev_nodes=15, tree="binary", name="step_b1_n15"),
        # a few users, 29 draft tokens (the paper's largest static tree) behind a tree of another size
        _case("step", 4, nodes=29, prev_nodes=16, tree="random", softplus=True, name="step_b4_n29"),
        # the benchmark's shape: 16 sequences, 64-node trees
        _case("step", 16, nodes=64, prev_nodes=64, tree="random", name="step_b16_n64"),
        # a full serving batch, beam of 3 x 16 tokens, state kept in bf16, raw step sizes, B and C in 8 groups
        _case("step", 64, groups=8, nodes=49, prev_nodes=49, tree="beam3", state="bf16", softplus=True,
              name="step_b64_n49_hb16"),
        # the widest beam of the paper (5 x 16 tokens): both trees above 64 nodes
        _case("step", 16, nodes=81, prev_nodes=81, tree="beam5", name="step_b16_n81"),
        # the fp32 configuration: 4 heads, 15 nodes, no conv
        _case("verify", 1, heads=4, dstate=64, dtype="f32", nodes=15, tree="binary", conv=False, name="verify_b1_n15_f32"),
        # the full layer in fp32, as a user runs it to check a model or where bf16 is not enough
        _case("verify", 4, dtype="f32", nodes=31, tree="binary", conv=True, name="verify_b4_n31_f32"),
        # the tree of the prefix-then-tree configuration
        _case("verify", 8, nodes=128, tree="random", conv=True, name="verify_b8_n128"),
        # the wide and deep tree configuration: 128 heads in 8 groups, 256 nodes
        _case("verify", 4, heads=128, groups=8, nodes=256, tree="random", conv=False, name="verify_b4_n256_g8"),
        # one user's prompt of odd length
        _case("prefill", 1, tokens=1013, want_y=True, h0=False, softplus=True, name="prefill_b1_t1013"),
        # the prefix of the prefix-then-tree configuration: the largest case
        _case("prefill", 8, tokens=4096, want_y=True, h0=False, name="prefill_b8_t4096"),
        # accepted text replayed into the state only, continuing from a state kept in bf16
        _case("prefill", 3, tokens=2050, want_y=False, h0=True, dstate=64, state="bf16", name="prefill_b3_t2050_state"),
    ]
    return cases


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))))


def draw(rng):
    """A case of the ranges above: batch 1 to 64, trees of 1 to 256 nodes, prompts of 16 to 4096 tokens."""
    kind = rng.choice(("step", "step", "verify", "verify", "prefill"))
    heads, headdim, dstate = rng.choice(((80, 64, 128), (80, 64, 128), (48, 64, 128), (24, 64, 128), (128, 64, 128),
                                         (80, 64, 64), (32, 64, 256), (40, 128, 128)))
    groups = rng.choice((1, 1, 8)) if heads % 8 == 0 else 1
    state = rng.choice(("f32", "f32", "bf16"))
    softplus = rng.random() < 0.4
    shape = dict(heads=heads, headdim=headdim, dstate=dstate, groups=groups, softplus=softplus)
    if kind == "prefill":
        tokens = _log_uniform(rng, 16, 4096)
        rows = 8 * 4096 * 80 * 64 * 128 // (heads * headdim * dstate)      # no dearer than the largest listed case
        batch = max(1, min(_log_uniform(rng, 1, 8), rows // tokens))
        return _case(kind, batch, state=state, tokens=tokens, want_y=rng.random() < 0.75, h0=rng.random() < 0.5, **shape)
    f32 = rng.random() < 0.2
    if f32:
        nodes = _log_uniform(rng, 1, 63)
        batch = max(1, min(_log_uniform(rng, 1, 4), 128 // nodes))
        shape.update(dtype="f32")
        state = "f32"
    elif kind == "step":
        nodes = _log_uniform(rng, 1, 100)
        batch = _log_uniform(rng, 1, 64)
    else:
        nodes = _log_uniform(rng, 1, 256)
        batch = max(1, min(_log_uniform(rng, 1, 16), 4 * 256 * 128 // (nodes * heads)))
    if dstate * headdim * heads > 80 * 64 * 128 or nodes > 64:
        batch = min(batch, 32)
    tree = rng.choice(("random", "random", "beam%d" % rng.randint(2, 5), "chain", "binary"))
    if kind == "step":
        prev = nodes if rng.random() < 0.5 else _log_uniform(rng, 1, 100 if nodes > 64 else 64)
        return _case(kind, batch, state=state, nodes=nodes, prev_nodes=prev, tree=tree, **shape)
    return _case(kind, batch, state=state, nodes=nodes, tree=tree, conv=rng.random() < 0.7, **shape)


# ---- inputs -------------------------------------------------------------------------------------------------------


def _one_tree(shape, n, g):
    if n == 1:
        return np.array([-1], dtype=np.int32)
    if shape == "chain":
        return synth.chain_tree(n)
    if shape == "binary":                              # filled level by level, the last level in part
        return synth.full_binary_tree(n.bit_length())[:n].copy()
    if shape.startswith("beam"):
        m = int(shape[4:])
        return synth.beam_tree(m, -(-(n - 1) // m), g)[:n].copy()
    depth, most = (min(n - 1, 4 + int(g.integers(0, 5))), 4) if n <= 128 else (10, 8)
    return synth.gen_tree(n, depth, most, g)


def _trees(shape, batch, n, g):
    return torch.from_numpy(np.stack([_one_tree(shape, n, g) for _ in range(batch)])).cuda()


def prepare(case, seed):
    c = case
    B, H, P, S, G = c["batch"], c["heads"], c["headdim"], c["dstate"], c["groups"]
    host = np.random.Generator(np.random.PCG64(seed))
    gen = torch.Generator(device="cuda").manual_seed(seed)
    io = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    Cc = H * P + 2 * G * S

    def normal(*shape, std=1.0, dtype=io):
        return torch.randn(shape, generator=gen, device="cuda").mul_(std).to(dtype)

    def uniform(lo, hi, *shape, dtype=io):
        return torch.rand(shape, generator=gen, device="cuda").mul_(hi - lo).add_(lo).to(dtype)

    def activations(rows):                             # what the conv and its SiLU leave: [B, rows, x | B | C]
        return torch.nn.functional.silu(torch.randn((B, rows, Cc), generator=gen, device="cuda").mul_(0.65)).to(io)

    def step_sizes(rows):                              # the raw projection, or the step size itself
        raw = torch.randn((B, rows, H), generator=gen, device="cuda")
        return raw if c["softplus"] else torch.nn.functional.softplus(raw - 2.0)

    s = dict(case=c, A=-torch.exp(uniform(0.0, 2.0, H, dtype=torch.float32)), D=normal(H, dtype=torch.float32),
             dt_bias=torch.full((H,), -2.0, device="cuda") if c["softplus"] else None,
             h0=normal(B, H, P, S, std=0.1, dtype=torch.bfloat16 if c["state"] == "bf16" else torch.float32))

    def columns(xbc):
        return (xbc[:, :, :H * P].unflatten(2, (H, P)), xbc[:, :, H * P:H * P + G * S].unflatten(2, (G, S)),
                xbc[:, :, H * P + G * S:].unflatten(2, (G, S)))

    if c["kind"] == "prefill":
        s["x"], s["Bm"], s["Cm"] = columns(activations(c["tokens"]))
        s["dt"] = step_sizes(c["tokens"])
        if not c["h0"]:
            s["h0"] = None
        return s
    N = c["nodes"]
    s["parent"] = _trees(c["tree"], B, N, host)
    s["dt"] = step_sizes(N)
    s["z"], s["norm_w"] = normal(B, N, H, P), uniform(0.5, 1.5, H * P)
    if c["kind"] == "step" or c["conv"]:
        s["xbc_pre"], s["conv_state"] = normal(B, N, Cc), normal(B, CONV_WIDTH - 1, Cc)
        s["conv_w"], s["conv_b"] = uniform(-0.5, 0.5, Cc, CONV_WIDTH), uniform(-0.5, 0.5, Cc)
    else:
        s["x"], s["Bm"], s["Cm"] = columns(activations(N))
    last = c["prev_nodes"] if c["kind"] == "step" else N
    s["accepted"] = torch.from_numpy(host.integers(0, last, size=B).astype(np.int32)).cuda()
    if c["kind"] == "step":
        s["prev_parent"] = _trees(c["tree"], B, last, host)
        s["prev_xbc_pre"], s["prev_xbc"], s["prev_dt"] = normal(B, last, Cc), activations(last), step_sizes(last)
    return s


# ---- one pass -----------------------------------------------------------------------------------------------------


def run(s):
    c = s["case"]
    H, P, S, G = c["heads"], c["headdim"], c["dstate"], c["groups"]
    if c["kind"] == "prefill":
        return st.stree_linear_ssd(s["x"], s["dt"], s["A"], s["Bm"], s["Cm"] if c["want_y"] else None,
                                   s["D"] if c["want_y"] else None, s["h0"], want_y=c["want_y"], dt_bias=s["dt_bias"])
    if c["kind"] == "step":
        y, h, xbc, conv_state = st.stree_tree_step(
            s["prev_parent"], s["accepted"], s["prev_xbc_pre"], s["prev_xbc"], s["prev_dt"], s["parent"], s["xbc_pre"],
            s["conv_state"], s["conv_w"], s["conv_b"], s["dt"], s["A"], s["D"], s["h0"], H, P, S, G,
            dt_bias=s["dt_bias"])
        out = st.stree_gate_norm(y, s["z"], s["norm_w"], G)
        return out, y, h, xbc, conv_state
    x, Bm, Cm, xbc, conv_in = s.get("x"), s.get("Bm"), s.get("Cm"), None, {}
    if c["conv"]:
        xbc = st.stree_tree_conv(s["parent"], s["xbc_pre"], s["conv_state"], s["conv_w"], s["conv_b"], H, P, S, G)
        x = xbc[:, :, :H * P].unflatten(2, (H, P))
        Bm = xbc[:, :, H * P:H * P + G * S].unflatten(2, (G, S))
        Cm = xbc[:, :, H * P + G * S:].unflatten(2, (G, S))
        conv_in = dict(xbc_pre=s["xbc_pre"], conv_state=s["conv_state"])
    y = st.stree_tree_ssd(s["parent"], x, s["dt"], s["A"], Bm, Cm, s["D"], s["h0"], dt_bias=s["dt_bias"])
    out = st.stree_gate_norm(y, s["z"], s["norm_w"], G)
    h, conv_state = st.stree_commit_state(s["parent"], s["accepted"], x, s["dt"], s["A"], Bm, s["h0"],
                                          dt_bias=s["dt_bias"], **conv_in)
    return out, y, h, xbc, conv_state


# ---- what a pass cannot do without, and how far two correct passes may be apart --------------------------------------


def work(case):
    c = case
    B, H, P, S, G, W = c["batch"], c["heads"], c["headdim"], c["dstate"], c["groups"], CONV_WIDTH
    e, es = (4 if c["dtype"] == "f32" else 2), (2 if c["state"] == "bf16" else 4)
    Cc, d, state = H * P + 2 * G * S, H * P, H * P * S * es
    if c["kind"] == "prefill":
        T, Q = c["tokens"], 64                          # flops: the chunked form, 64 tokens a chunk
        rows = T * ((2 * d + 2 * G * S) if c["want_y"] else (d + G * S)) * e + T * H * 4
        flops = H * T * 2 * P * S
        if c["want_y"]:
            flops += H * T * 2 * P * S + G * T * Q * S + H * T * Q * P
        return {"bytes": B * (rows + state * (2 if c["h0"] else 1)), "flops": B * flops}
    N = c["nodes"]
    path = 4 * (d + G * S) * e                          # x and B rows of an accepted path of a few nodes
    gate = N * d * e * 2                                # z read, result written (y is counted with the scan)
    scan = N * d * e + N * H * 4 + N * 4                # y written, dt, parents
    flops = G * N * (N + 1) * S + H * (N * (N + 1) * P + 2 * N * S * P)
    both_conv = 2 * N * Cc * e + 2 * (W - 1) * Cc * e   # rows before and behind the conv, both conv states
    if c["kind"] == "step":
        Np = c["prev_nodes"]
        total = both_conv + scan + gate + 2 * state + path + Np * (H * 4 + 4)
        return {"bytes": B * total + Cc * (W + 1) * e, "flops": B * (flops + N * Cc * 2 * W + 8 * H * P * S)}
    if c["conv"]:
        return {"bytes": B * (both_conv + scan + gate + 2 * state) + Cc * (W + 1) * e,
                "flops": B * (flops + N * Cc * 2 * W + 8 * H * P * S)}
    return {"bytes": B * (N * Cc * e + scan + gate + 2 * state), "flops": B * (flops + 8 * H * P * S)}


def tolerance(case):
    # Against the fp64 oracle: bf16 outputs are off by 1.7e-3 (conv, bf16 state) to 3.5e-3 (gated), fp32 ones by 1.5e-7
    # (2-norms).  Single values of the gated output are off by up to 0.22 of the rms: where a node's (dt <C,B> + D)
    # nearly cancels in a whole group, the norm scales that group's rounding up with it.
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.8}
