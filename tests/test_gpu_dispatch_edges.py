"""Edges of size rules: the smallest and odd row counts of the 2^15 inverse transform whose
workgroups walk the rows, the poly MAC on both sides of its rules for rows and loads, the
encoder with coefficients on both sides of 2^31, and rotations on both sides of the rule that
splits ModDown."""
import numpy as np
import pytest

from oracle import encode as OE
from oracle import linear as OL
from oracle import ntt as ON
from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("limbs,count", [(1, 1023), (1, 1024), (1, 1301), (3, 342), (2, 513)])
def test_intt_walk_n15(gpu_lib, limbs, count):
    import torch
    ck = gpu_lib
    ctx = ck.Context(15, limbs)
    n, qs = ctx.n, ctx.moduli
    g = torch.Generator(device="cuda:0")
    g.manual_seed(count)
    x = torch.empty((count, limbs, n), dtype=torch.int32, device="cuda:0")
    for l, q in enumerate(qs):
        x[:, l] = torch.randint(0, q, (count, n), dtype=torch.int32, device="cuda:0", generator=g)
    y = x.clone()
    ck.ckks_intt(ctx, y, count, limbs)
    for c in sorted({0, 255 // limbs, 256 // limbs, count - 1}):
        for l in range(limbs):
            want = ON.intt(ck.to_host_u32(x[c, l]), qs[l], ctx.roots[l], 15)
            assert np.array_equal(ck.to_host_u32(y[c, l]), want.astype(np.uint32))
    ck.ckks_ntt(ctx, y, count, limbs)
    assert torch.equal(x, y)
    ctx.close()


@pytest.mark.parametrize("log_n,limbs,d_out,d_in", [
    (14, 4, 27, 17), (14, 4, 28, 17), (14, 4, 29, 17), (14, 4, 30, 17), (14, 4, 32, 17), (14, 4, 33, 17),
    (14, 4, 32, 31), (14, 4, 32, 32),       # 2 groups of four rows a CU: below 256 MiB of plaintexts, and 256 MiB
    (14, 4, 31, 34), (14, 4, 48, 22),       # ragged, and 3 a CU
    (14, 4, 49, 21),                        # past 256 MiB, more than 3 a CU
    (14, 4, 28, 41), (14, 4, 28, 42),       # fewer than 2 a CU: below and past 288 MiB
    (14, 4, 49, 25),                        # past 288 MiB, more than 3 a CU
    (14, 16, 28, 3), (14, 16, 29, 3),       # 7 and 8 a CU
])
def test_mac_poly_rows_per_thread(gpu_lib, log_n, limbs, d_out, d_in):
    """Two rows a thread with plain and with non-temporal loads, and four rows, on both sides
    of every line between them."""
    import torch
    ck = gpu_lib
    ctx = ck.Context(log_n, limbs)
    qs, n = ctx.moduli, ctx.n
    g = torch.Generator(device="cuda:0")
    g.manual_seed(d_out * 100 + d_in)

    def uniform(*shape):
        x = torch.empty(shape + (limbs, n), dtype=torch.int32, device="cuda:0")
        for l, q in enumerate(qs):
            x[..., l, :] = torch.randint(0, q, shape + (n,), dtype=torch.int32, device="cuda:0", generator=g)
            x[..., l, 0] = q - 1                                # the largest sums
        return x

    pt, ct = uniform(d_out, d_in), uniform(d_in, 2)
    out = ck.empty_u32((d_out, 2, limbs, n))
    out.fill_(-1)
    ck.ckks_linear_mac_poly(ctx, pt, ct, out, d_out, d_in, limbs)
    rows = sorted({0, 1, d_out // 2, d_out - 3, d_out - 2, d_out - 1})
    want = OL.mac_poly(ck.to_host_u32(pt[rows]), ck.to_host_u32(ct), qs).astype(np.uint32)
    assert np.array_equal(ck.to_host_u32(out[rows]), want)
    ctx.close()


@pytest.mark.parametrize("log_n", [10, 11, 12, 13, 14])
@pytest.mark.parametrize("top", [2.0**29, 2.0**31 - 8, 2.0**31 + 8, 2.0**33])
def test_encode_coefficients_around_int32(gpu_lib, log_n, top):
    """The largest coefficient of random slots put at `top`, with both signs: int32 coefficients
    stay in registers, larger ones take the wide path.  Rounding ties aside the coefficients are
    the oracle's in every limb.  A tie: both sides' fp64 values, sums of N/2 terms, are within
    about sqrt(N/2) 2^-53 top of the exact one, so about N/2 * 2 sqrt(N/2) 2^-53 top of a
    vector's coefficients may round differently, by one; each shows four times (its mirror, and
    the vector with the other sign)."""
    ck = gpu_lib
    limbs = 3
    ctx = ck.Context(log_n, limbs)
    qs, psis, n = ctx.moduli, ctx.roots, ctx.n
    z = gen.poly_weights(np.random.default_rng(log_n), 1, 1, n // 2)[0]
    z = np.concatenate([z, -z, z[:, ::-1] * 1e-3])
    m = OE.encode_coeffs(z, log_n)
    scale = top / np.max(np.abs(m))
    want = OE.round_coeffs(m, scale)
    assert abs(np.max(np.abs(want)) - top) <= 1
    ties = n / 2 * 2 * np.sqrt(n / 2) * 2.0**-53 * top
    most = 4 * (1 + ties + 3 * np.sqrt(ties))
    pt = ck.empty_u32((3, limbs, n))
    pt.fill_(-1)
    ck.ckks_linear_encode_poly(ctx, ck.to_device(np.ascontiguousarray(z)), 3, limbs, scale, pt)
    got = ck.to_host_u32(pt)
    for l, q in enumerate(qs):
        assert got[:, l].max() < q
        coef = ON.intt(got[:, l], q, psis[l], log_n).astype(np.int64)
        diff = np.mod(coef - np.mod(want, q).astype(np.int64), q)
        off = diff != 0
        assert np.all((diff[off] == 1) | (diff[off] == q - 1)) and off.sum() <= most, (l, off.sum(), most)
    ctx.close()


@pytest.mark.parametrize("log_n,L,count,small,two", [
    (10, 4, 128, 127, False), (11, 5, 97, 48, False),                          # few points of transforms to save
    (13, 5, 96, 95, True), (14, 3, 192, 100, True),                            # three workgroups a CU, and fewer
    (10, 5, 384, 383, True), (11, 4, 288, 287, True), (12, 3, 288, 287, True)])  # just as many points, and fewer
@pytest.mark.parametrize("hoisted", [True, False])
def test_many_rotations_equal_few(gpu_lib, log_n, L, count, small, two, hoisted):
    """A batch of rotations whose ModDown takes two launches (`two`) or one against the same
    rotations in smaller calls of one launch, which the oracle covers."""
    ck = gpu_lib
    ctx = ck.Context(log_n, L)
    n, lk, qs = ctx.n, L - 1, ctx.moduli
    in_two = [2 * c * lk >= 3 * 256 and 2 * c * (lk - 1) * n >= 9216 * 256 for c in (count, small)]
    assert in_two == [two, False]
    rng = np.random.default_rng(log_n * 100 + count)
    ct = ck.to_device(gen.uniform_residues(rng, (1 if hoisted else count, 2), qs[:lk], n))
    ksk = ck.to_device(gen.uniform_residues(rng, (count, lk, 2), qs, n))
    got, ref = ck.empty_u32((count, 2, lk, n)), ck.empty_u32((count, 2, lk, n))
    got.fill_(-1)
    ws = ck.empty_workspace(ck.rotate_workspace_bytes(ctx, count, hoisted))
    ck.ckks_rotate(ctx, ct, count, 3, 5, hoisted, ksk, ws, got)
    for k in range(0, count, small):
        m = min(small, count - k)
        ck.ckks_rotate(ctx, ct if hoisted else ct[k:k + m], m, 3 + 5 * k, 5, hoisted, ksk[k:k + m], ws, ref[k:k + m])
    assert np.array_equal(ck.to_host_u32(got), ck.to_host_u32(ref))
    ctx.close()
