"""The work that users of the library have it do, as cases that can be timed.

A case is a dict of plain values.  `prepare` makes what a caller has in hand
before a call (context, inputs, keys, output buffers, workspace), `run` makes
one pass through the public entry points and returns the whole outputs.

Kinds:
  scalar   one projection layer with scalar weights: ckks_linear_encode_scalar,
           ckks_linear_mac_scalar, ckks_rescale
  poly     one layer with full-polynomial weights encoded on the call:
           ckks_linear_encode_poly, ckks_linear_mac_poly, ckks_rescale
  stack    a decode stack of full-polynomial groups run by planner.Executor:
           part of the weights resident, part encoded on the call, rescale and
           refresh between the groups
  ntt      ckks_ntt of one batch and ckks_intt of another
  refresh  ckks_refresh, decrypt-then-encrypt of a layer's outputs
  client   the trusted side around a call: ckks_linear_encode_poly,
           ckks_encrypt, ckks_decrypt
  bsgs     ckks_linear_bsgs, the diagonal matrix-vector product with rotations

Every output is a residue below its prime with one right value, so all cases
are compared exactly.
"""
from __future__ import annotations

import math

import torch

import paper_2606_17421_amd as ck
from paper_2606_17421_amd.planner import Executor, LinearGroup, plan

WEIGHT_STD = 0.02       # trained projection weights are about this wide
ERROR_SIGMA = 3.2       # RLWE error, clipped to six sigma
ERROR_BOUND = 19


def listed():
    return [
        # The smallest layer: 16 features in a ring of 2^10; launches and latency.
        dict(name="layer-16-n10", kind="scalar", log_n=10, limbs=2, log_scale=25, d_in=16, d_out=16),
        # GPT-2-124M attention output projection.
        dict(name="layer-768x768-n14", kind="scalar", log_n=14, limbs=4, log_scale=26, d_in=768, d_out=768),
        # GPT-2-124M FFN up projection, and a down projection (deep contraction, few outputs).
        dict(name="layer-768x3072-n15", kind="scalar", log_n=15, limbs=6, log_scale=26, d_in=768, d_out=3072),
        dict(name="layer-3072x768-n14", kind="scalar", log_n=14, limbs=4, log_scale=26, d_in=3072, d_out=768),
        # Qwen3-0.6B gate and up projections stacked: the largest layer.
        dict(name="layer-1024x6144-n16", kind="scalar", log_n=16, limbs=8, log_scale=28, d_in=1024, d_out=6144),
        # Weights that do not stay resident: encoded as full polynomials on every call.
        dict(name="poly-64x64-n15", kind="poly", log_n=15, limbs=6, log_scale=30, d_in=64, d_out=64),
        # Four decode layers of (QKV, O, GateUp, Down) groups, 13 of the 16 groups resident.
        dict(name="stack-4-layers-n14", kind="stack", log_n=14, limbs=4, log_scale=26, d=32, layers=4, pinned=13),
        # Standalone transforms of every output polynomial of the 768 -> 3072 layer.
        dict(name="ntt-36864-n15", kind="ntt", log_n=15, limbs=6, count=6144),
        # Refresh of a 768-feature layer's rescaled outputs back to the full chain.
        dict(name="refresh-768-n14", kind="refresh", log_n=14, limbs=4, limbs_in=3, count=768),
        # The trusted side of a call at the largest ring: encode, encrypt, decrypt 100 features.
        dict(name="client-100-n16", kind="client", log_n=16, limbs=8, log_scale=28, count=100),
        # A 1024 x 1024 product by diagonals and rotations: one vector (decode), and a batch.
        dict(name="bsgs-1024-n13", kind="bsgs", log_n=13, limbs=4, log_scale=26, n1=32, n2=32, count=1),
        dict(name="bsgs-1024-n13-x16", kind="bsgs", log_n=13, limbs=4, log_scale=26, n1=32, n2=32, count=16),
    ]


def _spread(rng, lo, hi):
    """A whole number in [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def _draw_once(rng):
    kind = rng.choice(["scalar", "scalar", "scalar", "poly", "stack", "ntt", "refresh", "client", "bsgs"])
    c = dict(kind=kind)
    if kind == "scalar":
        c.update(log_n=rng.randint(10, 16), limbs=rng.randint(2, 8), log_scale=rng.randint(25, 28),
                 d_in=_spread(rng, 16, 3072), d_out=_spread(rng, 16, 6144))
    elif kind == "poly":
        c.update(log_n=rng.randint(12, 16), limbs=rng.randint(2, 6), log_scale=rng.randint(26, 30),
                 d_in=_spread(rng, 4, 96), d_out=_spread(rng, 4, 96))
    elif kind == "stack":
        layers = rng.randint(1, 4)
        c.update(log_n=rng.randint(12, 14), limbs=rng.randint(4, 6), log_scale=26, d=_spread(rng, 8, 48),
                 layers=layers, pinned=rng.randint(0, 4 * layers))
    elif kind == "ntt":
        c.update(log_n=rng.randint(10, 16), limbs=rng.randint(1, 8), count=_spread(rng, 1, 6144))
    elif kind == "refresh":
        c.update(log_n=rng.randint(11, 16), limbs=rng.randint(3, 8), limbs_in=rng.randint(2, 3),
                 count=_spread(rng, 1, 1024))
    elif kind == "client":
        c.update(log_n=rng.randint(11, 16), limbs=rng.randint(2, 8), log_scale=rng.randint(25, 30),
                 count=_spread(rng, 1, 768))
    else:
        n1 = rng.choice([8, 16, 32])
        c.update(log_n=rng.randint(11, 14), limbs=rng.randint(3, 4), log_scale=26, n1=n1,
                 n2=rng.choice([n1, n1 // 2, n1 - 3]), count=_spread(rng, 1, 32))
    return c


def draw(rng):
    while True:
        c = _draw_once(rng)
        w = work(c)
        # well below the largest listed case in memory traffic and in operations
        if w["bytes"] <= 8e9 and w["flops"] <= 4e12 and _state_bytes(c) <= 20e9:
            return c


def _state_bytes(c):
    n, L = 1 << c["log_n"], c["limbs"]
    k = c["kind"]
    if k == "scalar":
        return 4 * n * 2 * (L * (c["d_in"] + c["d_out"]) + (L - 1) * c["d_out"])
    if k == "poly":
        return 4 * n * (L + 1) * c["d_in"] * c["d_out"] + 16 * n * L * (c["d_in"] + c["d_out"])
    if k == "bsgs":
        return 4 * n * (c["n1"] * c["n2"] * L + c["count"] * (c["n1"] + c["n2"]) * 8 * (L + 1) * (L + 1))
    if k == "stack":
        return 4 * c["layers"] * c["d"] ** 2 * n * 4 * (L + 1)
    return 4 * n * c["count"] * 8 * L


def _butterflies(n, rows):
    return rows * (n // 2) * (n.bit_length() - 1)


def work(case):
    """Bytes: every input read once, every output written once.  Operations: two
    per modular multiply-add, three per butterfly of a transform (a modular
    product, a sum and a difference), five N log N for the encoder's real
    spectral transform."""
    c, k = case, case["kind"]
    n, L = 1 << c["log_n"], c["limbs"]
    row = 4 * n                                       # bytes of one limb row

    def rescale_ops(cts, limbs):                      # one inverse, limbs - 1 forward transforms, the combine
        return 3 * _butterflies(n, 2 * cts * limbs) + 4 * n * cts * (limbs - 1)

    def encode_ops(polys, limbs):
        return polys * 5 * (n // 2) * c["log_n"] + 3 * _butterflies(n, polys * limbs)

    def refresh_ops(cts, limbs_out):
        return 3 * _butterflies(n, cts * (2 + limbs_out)) + 2 * n * cts * (2 + limbs_out)

    if k == "scalar":
        i, o = c["d_in"], c["d_out"]
        return {"bytes": 2 * row * (L * i + (L - 1) * o) + 8 * i * o,
                "flops": 4 * i * o * L * n + rescale_ops(o, L)}
    if k == "poly":
        i, o = c["d_in"], c["d_out"]
        return {"bytes": 4 * n * i * o + 2 * row * (L * i + (L - 1) * o),
                "flops": encode_ops(i * o, L) + 4 * i * o * L * n + rescale_ops(o, L)}
    if k == "stack":
        p, d = _stack_plan(c), c["d"]
        b, f = 2 * row * d * L, 0
        for s in p.steps:
            b += s.encoded_bytes if s.pinned else 4 * n * d * d
            f += 4 * d * d * s.level * n + rescale_ops(d, s.level) + (0 if s.pinned else encode_ops(d * d, s.level))
            if s.refresh_after:
                b += d * (L * row + 4 * n)            # the fresh a and e
                f += refresh_ops(d, L)
        return {"bytes": b + 2 * row * d * (p.steps[-1].level - 1), "flops": f}
    if k == "ntt":
        rows = c["count"] * L
        return {"bytes": 4 * row * rows, "flops": 6 * _butterflies(n, rows)}
    if k == "refresh":
        m = c["count"]
        return {"bytes": row * m * (4 + L + 1 + 2 * L), "flops": refresh_ops(m, L)}
    if k == "client":
        m = c["count"]
        return {"bytes": m * (4 * n + L * row + 4 * n + 3 * L * row + L * row),
                "flops": encode_ops(m, L) + 3 * _butterflies(n, 2 * m * L) + 4 * n * m * L}
    n1, n2, m = c["n1"], c["n2"], c["count"]
    keys = n1 + n2 - 2
    lp = L + 1
    ops = 4 * m * n1 * n2 * L * n                     # the inner sums
    ops += m * keys * 4 * L * lp * n                  # key-switching inner products
    # ModUp of the input and of n2 - 1 sums, ModDown of n1 - 1 rotations and of the sum, the closing rescale
    ops += m * 3 * _butterflies(n, n2 * L * (1 + L) + (n1 - 1) * 2 * lp + 2 * lp + 2 * L)
    return {"bytes": n1 * n2 * L * row + keys * L * 2 * lp * row + m * 2 * row * (L + L - 1), "flops": ops}


def tolerance(case):
    """Residues are whole numbers with one right value."""
    return "exact"


def exact(case, seed):
    """No output is a floating-point number: there is nothing to evaluate more precisely."""
    return None


# ---- inputs -----------------------------------------------------------------

def _gen(seed, salt=0):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(2606 * 1000003 + 7919 * seed + salt)
    return g


def _uniform(g, prefix, moduli, n):
    """int32 prefix + (limbs, n): limb l uniform in [0, q_l)."""
    out = torch.empty(tuple(prefix) + (len(moduli), n), dtype=torch.int32, device="cuda:0")
    for l, q in enumerate(moduli):
        out[..., l, :] = torch.randint(0, int(q), tuple(prefix) + (n,), dtype=torch.int32, device="cuda:0", generator=g)
    return out


def _normal(g, shape, std):
    return torch.randn(shape, dtype=torch.float64, device="cuda:0", generator=g) * std


def _errors(g, shape):
    e = torch.randn(shape, dtype=torch.float32, device="cuda:0", generator=g) * ERROR_SIGMA
    return e.round_().clamp_(-ERROR_BOUND, ERROR_BOUND).to(torch.int32)


def _secret(g, ctx):
    """A ternary secret, NTT form under every prime of the context."""
    s = torch.randint(-1, 2, (ctx.n,), dtype=torch.int64, device="cuda:0", generator=g)
    q = torch.tensor(ctx.moduli, dtype=torch.int64, device="cuda:0")
    s_ntt = torch.remainder(s[None, :], q[:, None]).to(torch.int32).contiguous()
    ck.ckks_ntt(ctx, s_ntt, 1, ctx.limbs)
    return s_ntt


def _workspace(nbytes):
    return ck.empty_workspace(nbytes)


def _stack_plan(c):
    groups = []
    for i in range(c["layers"]):
        for name, tee in (("qkv", True), ("o", False), ("gateup", True), ("down", True)):
            groups.append(LinearGroup(f"l{i}.{name}", c["d"], c["d"], tee_after=tee))
    n, L = 1 << c["log_n"], c["limbs"]
    every = plan(groups, 1 << 62, L, n)
    return plan(groups, sum(s.encoded_bytes for s in every.steps[:c["pinned"]]), L, n)


def prepare(case, seed):
    c, k = case, case["kind"]
    L = c["limbs"]
    g = _gen(seed)
    ctx = ck.Context(c["log_n"], L + 1 if k == "bsgs" else L)
    n = ctx.n
    st = dict(c, ctx=ctx)
    scale = float(1 << c["log_scale"]) if "log_scale" in c else None
    st["scale"] = scale
    if k == "scalar":
        i, o = c["d_in"], c["d_out"]
        st["w"] = _normal(g, (o, i), WEIGHT_STD)
        st["ct"] = _uniform(g, (i, 2), ctx.moduli, n)
        st["w_enc"] = ck.empty_u32((o, i, L))
        st["mac"] = ck.empty_u32((o, 2, L, n))
        st["out"] = ck.empty_u32((o, 2, L - 1, n))
        st["mac_ws"] = _workspace(ck.ckks_workspace_bytes(ctx, ck.CKKS_OP_MAC_SCALAR, o, i, L))
        st["ws"] = _workspace(ck.ckks_workspace_bytes(ctx, ck.CKKS_OP_RESCALE, o, 0, L))
    elif k == "poly":
        i, o = c["d_in"], c["d_out"]
        st["slots"] = _normal(g, (o * i, n // 2), WEIGHT_STD)
        st["ct"] = _uniform(g, (i, 2), ctx.moduli, n)
        st["pt"] = ck.empty_u32((o, i, L, n))
        st["mac"] = ck.empty_u32((o, 2, L, n))
        st["out"] = ck.empty_u32((o, 2, L - 1, n))
        st["ws"] = _workspace(ck.ckks_workspace_bytes(ctx, ck.CKKS_OP_RESCALE, o, 0, L))
    elif k == "stack":
        p, d = _stack_plan(c), c["d"]
        weights = [_normal(g, (d * d, n // 2), WEIGHT_STD) for _ in p.steps]
        st["ex"] = Executor(ctx, p, weights, scale, _secret(g, ctx))
        st["ct"] = _uniform(g, (d, 2), ctx.moduli, n)
        st["draws"] = [(_uniform(g, (d,), ctx.moduli, n), _errors(g, (d, n))) for _ in range(p.refreshes)]
    elif k == "ntt":
        st["fwd"] = _uniform(g, (c["count"],), ctx.moduli, n)
        st["inv"] = _uniform(g, (c["count"],), ctx.moduli, n)
    elif k == "refresh":
        m = c["count"]
        st["s"] = _secret(g, ctx)
        st["ct"] = _uniform(g, (m, 2), ctx.moduli[:c["limbs_in"]], n)
        st["a"] = _uniform(g, (m,), ctx.moduli, n)
        st["e"] = _errors(g, (m, n))
        st["out"] = ck.empty_u32((m, 2, L, n))
    elif k == "client":
        m = c["count"]
        st["s"] = _secret(g, ctx)
        st["slots"] = torch.rand((m, n // 2), dtype=torch.float64, device="cuda:0", generator=g) * 2 - 1
        st["a"] = _uniform(g, (m,), ctx.moduli, n)
        st["e"] = _errors(g, (m, n))
        st["pt"] = ck.empty_u32((m, L, n))
        st["ct"] = ck.empty_u32((m, 2, L, n))
        st["m"] = ck.empty_u32((m, L, n))
    else:
        n1, n2, m = c["n1"], c["n2"], c["count"]
        s = _secret(g, ctx)
        slots = _normal(g, (n2 * n1, n // 2), WEIGHT_STD)
        st["pt"] = ck.empty_u32((n2, n1, L, n))
        ck.ckks_linear_encode_poly(ctx, slots, n2 * n1, L, scale, st["pt"])
        words = L * 2 * (L + 1) * n
        st["ksk"] = ck.empty_u32(((n1 + n2 - 2) * words,))
        for r0, cnt, off in ((1, n1 - 1, 0), (n1, n2 - 1, n1 - 1)):
            if cnt:
                ck.ckks_keygen_rotation(ctx, s, r0, r0, cnt, _uniform(g, (cnt, L), ctx.moduli, n),
                                        _errors(g, (cnt, L, n)), st["ksk"][off * words:(off + cnt) * words])
        st["ct"] = ck.empty_u32((m, 2, L, n))
        x = torch.rand((m, n // 2), dtype=torch.float64, device="cuda:0", generator=g) * 2 - 1
        px = ck.empty_u32((m, L, n))
        ck.ckks_linear_encode_poly(ctx, x, m, L, scale, px)
        ck.ckks_encrypt(ctx, px, s[:L].contiguous(), _uniform(g, (m,), ctx.moduli[:L], n), _errors(g, (m, n)), m, L,
                        st["ct"])
        st["out"] = ck.empty_u32((m, 2, L - 1, n))
        st["ws"] = _workspace(ck.bsgs_workspace_bytes(ctx, m, n1, n2))
    return st


def run(state):
    s, k, ctx, L = state, state["kind"], state["ctx"], state["limbs"]
    if k == "scalar":
        i, o = s["d_in"], s["d_out"]
        ck.ckks_linear_encode_scalar(ctx, s["w"], o, i, L, s["scale"], s["w_enc"])
        ck.ckks_linear_mac_scalar(ctx, s["w_enc"], s["ct"], s["mac"], o, i, L, s["mac_ws"])
        ck.ckks_rescale(ctx, s["mac"], s["out"], o, L, s["ws"])
        return s["out"], s["w_enc"]
    if k == "poly":
        i, o = s["d_in"], s["d_out"]
        ck.ckks_linear_encode_poly(ctx, s["slots"], o * i, L, s["scale"], s["pt"])
        ck.ckks_linear_mac_poly(ctx, s["pt"], s["ct"], s["mac"], o, i, L)
        ck.ckks_rescale(ctx, s["mac"], s["out"], o, L, s["ws"])
        return s["out"], s["pt"]
    if k == "stack":
        out, limbs = s["ex"].run(s["ct"], s["draws"])
        return out, limbs
    if k == "ntt":
        ck.ckks_ntt(ctx, s["fwd"], s["count"], L)
        ck.ckks_intt(ctx, s["inv"], s["count"], L)
        return s["fwd"], s["inv"]
    if k == "refresh":
        ck.ckks_refresh(ctx, s["ct"], s["limbs_in"], s["s"], s["a"], s["e"], s["count"], L, s["out"])
        return s["out"]
    if k == "client":
        ck.ckks_linear_encode_poly(ctx, s["slots"], s["count"], L, s["scale"], s["pt"])
        ck.ckks_encrypt(ctx, s["pt"], s["s"], s["a"], s["e"], s["count"], L, s["ct"])
        ck.ckks_decrypt(ctx, s["ct"], s["s"], s["count"], L, s["m"])
        return s["ct"], s["m"], s["pt"]
    ck.ckks_linear_bsgs(ctx, s["pt"], s["ct"], s["count"], s["n1"], s["n2"], s["ksk"], s["ws"], s["out"])
    return s["out"]
