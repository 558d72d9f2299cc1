"""The residue-channel form of the scalar MAC (csrc/mac_rns.hip): its arithmetic on the
CPU, and the kernels against the vector MAC and the oracle at the edges of what it takes."""
import math

import numpy as np
import pytest

from oracle import linear as OL
from workloads import gen

MODULI = (256, 247, 245, 243, 241, 239, 233, 229)
M = math.prod(MODULI)
ROW_LIMIT = int(0.46 * M / 2**29)      # largest sum |v| of a row that the kernels take
OFFSET = 1 << 29


def test_moduli_are_coprime_and_the_row_limit_covers_scaled_weights():
    for i, a in enumerate(MODULI):
        for b in MODULI[:i]:
            assert math.gcd(a, b) == 1
    assert all(m <= 247 or m == 256 for m in MODULI)
    # 1024 weights N(0, 0.02^2) at scale 2^28, six standard deviations above the mean row sum
    sd = 0.02 * 2**28
    assert 1024 * 0.798 * sd + 6 * 0.603 * sd * 32 < ROW_LIMIT


def test_operand_bytes():
    """The operand byte of u (for u - 2^29, times w) is an int8 in the right class."""
    rng = np.random.default_rng(5)
    u = np.concatenate([rng.integers(0, 1 << 30, 200000), [0, 1, OFFSET - 1, OFFSET, OFFSET + 1, (1 << 30) - 1]])
    for m in MODULI:
        for w in (1, pow(M // m % m, -1, m)):
            y = sum(((u >> (8 * b)) & 255) * (w * 256**b % m) for b in range(4)) + 128 + (-OFFSET * w) % m
            assert y.max() < 1 << 18
            q = (y * -(-(1 << 32) // m)) >> 32
            byte = y - q * m - 128
            assert np.array_equal(q, y // m)
            assert byte.min() >= -128 and byte.max() <= 127
            assert not ((byte - (u - OFFSET) * w) % m).any()


def test_channel_reduction_gives_bytes():
    """s - mulhi(s, floor(2^32 / m)) m lies in [0, 255] for every biased sum s < 2^27 + 2^8."""
    rng = np.random.default_rng(6)
    for m in MODULI:
        bias = ((1 << 26) // m + 1) * m
        assert bias >= 1 << 26                                    # 4096 products of two int8
        s = np.concatenate([rng.integers(0, (1 << 27) + 256, 200000), np.arange(bias + (1 << 26) - 4 * m, bias + (1 << 26) + 1),
                            np.arange(0, 4 * m)])
        r = s - ((s * ((1 << 32) // m)) >> 32) * m
        assert r.min() >= 0 and r.max() <= 255 and not ((r - s) % m).any()


@pytest.mark.parametrize("q", [(1 << 30) - 35, 536903681])
def test_combination_is_exact_up_to_the_limit(q):
    """sum r_k C_k - alpha M from bytes, for |T| up to 0.46 M and any representatives of the residues."""
    rng = np.random.default_rng(7)
    top = ROW_LIMIT * OFFSET
    c = [M // m % q for m in MODULI]
    f = [((1 << 16) // m + 1) // 2 for m in MODULI]
    cases = [0, 1, -1, top, -top, top - 1, 1 - top] + [int(x * top) for x in rng.uniform(-1, 1, 3000)]
    for t in cases:
        for lift in (0, 1, 2):
            r = []
            for k, m in enumerate(MODULI):
                x = t * pow(M // m, -1, m) % m
                r.append(x + m if x + m <= 254 and (lift == 1 or (lift == 2 and rng.integers(2))) else x)
            alpha = (sum(a * b for a, b in zip(r, f)) + (1 << 14)) >> 15
            assert sum(x * (M // m) for x, m in zip(r, MODULI)) - alpha * M == t
            v = sum(a * b for a, b in zip(r, c)) + alpha * ((q - M % q) % q) + q - 1   # q - 1: the largest row constant
            assert v < 1 << 45
            qt = ((v >> 16) * ((1 << 48) // q)) >> 32
            assert 0 <= v - qt * q < 2 * q


TAKEN = 0x524E5301                     # the decision word of a call that the channels computed


def _weights(kind, rng, d_out, d_in, qs):
    """Per-limb residues of centred integers (d_out, d_in)."""
    if kind in ("row-limit", "above-row-limit"):     # every row sum at the limit, signs by row
        v = np.full((d_out, d_in), ROW_LIMIT // d_in, dtype=np.int64) * np.where(np.arange(d_out) % 2, 1, -1)[:, None]
        if kind == "above-row-limit":                # one row whose sums reach 0.6 M: the channels would lose them
            v[d_out // 2] = int(0.6 * M / 2**29 / d_in)
    else:
        v = np.rint(gen.scalar_weights(rng, d_out, d_in) * 2.0 ** (26 if kind == "three-digit" else 28)).astype(np.int64)
        if isinstance(kind, int):                    # `kind` 16-row tiles of four digits, from the last tile on
            v = np.clip(v, -0x7F7F7F, 0x7F7F7F)
            v[[d_out - 1 - 16 * k for k in range(kind)], d_in - 1] = 0x808080
    w = np.stack([np.mod(v, q).astype(np.uint32) for q in qs], -1)
    if kind == "one-limb-differs":
        w[d_out - 1, d_in - 1, len(qs) - 1] = (w[d_out - 1, d_in - 1, len(qs) - 1] + 1) % qs[-1]
    return w


def _residues(ck, ctx, d_in, seed):
    """Residues 0 or q - 1 in half of the columns (the largest sums), uniform in the others."""
    import torch
    n, qs = ctx.n, ctx.moduli
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    ct = torch.empty((d_in, 2, len(qs), n), dtype=torch.int32, device="cuda:0")
    for l, q in enumerate(qs):
        ct[:, :, l] = torch.randint(0, q, (d_in, 2, n), dtype=torch.int32, device="cuda:0", generator=g)
        ct[:, :, l, 1::2] = torch.where(torch.rand((d_in, 2, n // 2), device="cuda:0", generator=g) < 0.5, 0, q - 1).to(torch.int32)
    ct[:, :, :, 3] = 0
    ct[:, :, :, 5] = torch.tensor([q - 1 for q in qs], dtype=torch.int32, device="cuda:0")
    return ct


def _took_channels(ck, ws, d_out, d_in, limbs):
    """Whether the last call on this workspace left the channels' decision word, which lies
    behind the digit fragments (the digit split writes a tile flag, 0 or 1, there)."""
    at = limbs * (-(-d_out // 128) * 8) * -(-d_in // 64) * 4096 // 4
    word = int(ck.to_host_u32(ws.view(-1)[at:at + 1].clone())[0])
    assert word in (0, 1, TAKEN)
    return word == TAKEN


def _check(ck, ctx, w, ct, ws, d_out, d_in, taken):
    import torch
    L, n, qs = ctx.limbs, ctx.n, ctx.moduli
    d_w = ck.to_device(w)
    got, ref = ck.empty_u32((d_out, 2, L, n)), ck.empty_u32((d_out, 2, L, n))
    got.fill_(-1)
    ck.ckks_linear_mac_scalar(ctx, d_w, ct, got, d_out, d_in, L, ws)
    assert _took_channels(ck, ws, d_out, d_in, L) == taken
    ck.ckks_ctx_set_mac_algo(ctx, ck.CKKS_MAC_VALU)
    ck.ckks_linear_mac_scalar(ctx, d_w, ct, ref, d_out, d_in, L)
    ck.ckks_ctx_set_mac_algo(ctx, ck.CKKS_MAC_AUTO)
    assert torch.equal(got, ref)
    cols = [0, 1, 3, 5, 127, 128, n - 1]
    rows = [0, 255, 256, d_out - 1]
    want = OL.mac_scalar(w, ck.to_host_u32(ct[..., cols].contiguous()), qs, rows=rows).astype(np.uint32)
    assert np.array_equal(ck.to_host_u32(got[rows][..., cols].contiguous()), want)


@pytest.mark.gpu
@pytest.mark.parametrize("kind,log_n,L,d_out,d_in,taken", [
    ("encoded", 14, 8, 8191, 1000, True),   # last row block 255 rows deep, last k-step 40 deep, ragged chunk of strips
    ("encoded", 14, 8, 8193, 1024, True),    # one row in the last block
    ("encoded", 14, 12, 7167, 950, True),   # an odd number of k-steps
    ("row-limit", 14, 8, 8191, 1000, True),
    # refused by the weights
    ("above-row-limit", 14, 8, 8191, 1000, False),
    ("one-limb-differs", 14, 8, 8191, 1000, False),
    ("three-digit", 14, 8, 8191, 1000, False),
    (224, 14, 12, 7167, 1000, True),         # half of the 448 row tiles of four digits, and one less
    (223, 14, 12, 7167, 1000, False),
    # refused by the shape, slower in the channels: few rounds of workgroups a chunk, a padded
    # last row block, a shallow contraction
    ("encoded", 14, 16, 2303, 1000, False),
    ("encoded", 14, 16, 2049, 1024, False),
    ("encoded", 14, 16, 4200, 513, False),
    ("encoded", 13, 16, 17000, 256, False),
])
def test_large_layer_matches_the_vector_mac(gpu_lib, kind, log_n, L, d_out, d_in, taken):
    """At least 2^40 products, where the residue-channel kernels may be tried: which kernels
    ran, the whole output against the vector kernel, and sampled rows and columns against the
    oracle."""
    ck = gpu_lib
    ctx = ck.Context(log_n, L)
    assert d_out * d_in * 2 * L * ctx.n >= 1 << 40
    w = _weights(kind, np.random.default_rng(d_out + d_in), d_out, d_in, ctx.moduli)
    ct = _residues(ck, ctx, d_in, d_out * 31 + d_in)
    ws = ck.empty_workspace(ck.ckks_workspace_bytes(ctx, ck.CKKS_OP_MAC_SCALAR, d_out, d_in, L))
    ws.random_()
    _check(ck, ctx, w, ct, ws, d_out, d_in, taken)
    ctx.close()


@pytest.mark.gpu
def test_one_workspace_for_both_forms(gpu_lib):
    """Taken, refused and taken again on one workspace: a call's decision word and planes are
    what the next one finds where its tile flags and fragments go."""
    ck = gpu_lib
    ctx = ck.Context(14, 8)
    d_out, d_in = 8191, 1000
    ct = _residues(ck, ctx, d_in, 8)
    ws = ck.empty_workspace(ck.ckks_workspace_bytes(ctx, ck.CKKS_OP_MAC_SCALAR, d_out, d_in, 8))
    for kind in ("encoded", "three-digit", "row-limit", "one-limb-differs"):
        w = _weights(kind, np.random.default_rng(9), d_out, d_in, ctx.moduli)
        _check(ck, ctx, w, ct, ws, d_out, d_in, kind in ("encoded", "row-limit"))
    ctx.close()
