"""Encryption and decryption below and above one row per CU, with one limb, at the largest
whole-row ring and in the staged 2^16 form, each with and without a plaintext, against the
oracle bit for bit; the refresh at the ends of the error range."""
import numpy as np
import pytest

from oracle import rlwe as OR
from test_gpu_rlwe import setup, residues_of
from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("log_n,limbs,count", [(13, 5, 51), (13, 4, 64), (14, 3, 85), (14, 4, 65), (15, 2, 3), (12, 1, 9), (16, 1, 3)])
@pytest.mark.parametrize("with_pt", [True, False])
def test_rows_match_the_oracle(gpu_lib, log_n, limbs, count, with_pt):
    ck = gpu_lib
    ctx, qs, psis, n, st, s, s_ntt, m, e, a = setup(ck, log_n, limbs, count, 900 + log_n + limbs)
    if not with_pt:
        m = np.zeros_like(m)
    # the extremes of the error range of every limb, |e| < q_l
    e[0, :4] = [min(qs) - 1, 1 - min(qs), 0, -1]
    pt = None
    if with_pt:
        pt = ck.to_device(residues_of(m, qs))
        ck.ckks_ntt(ctx, pt, count, limbs)
    ct = ck.empty_u32((count, 2, limbs, n))
    ct.fill_(-1)
    ck.ckks_encrypt(ctx, pt, s_ntt, ck.to_device(a), ck.to_device(e), count, limbs, ct)
    pick = sorted({0, count // 2, count - 1})
    got = ck.to_host_u32(ct)[pick]
    want = OR.encrypt(m[pick], s, a[pick], e[pick], qs, psis, log_n).astype(np.uint32)
    assert np.array_equal(got, want)
    out = ck.empty_u32((count, limbs, n))
    out.fill_(-1)
    ck.ckks_decrypt(ctx, ct, s_ntt, count, limbs, out)
    # an encryption of m with error e decrypts to m + e in every limb
    assert np.array_equal(ck.to_host_u32(out), residues_of(m + e, qs))


@pytest.mark.parametrize("log_n,limbs,count", [(10, 3, 2), (13, 2, 2), (13, 4, 65), (14, 3, 2), (15, 2, 1), (16, 2, 1)])
def test_refresh_with_errors_up_to_the_prime(gpu_lib, log_n, limbs, count):
    """|e| < q_l in every limb, the extremes on coefficients of every size: residues of a
    uniform ciphertext, in the fused, two-kernel and staged forms."""
    ck = gpu_lib
    ctx, qs, psis, n, st, s, s_ntt, m, e, a = setup(ck, log_n, limbs, count, 950 + log_n)
    ct = gen.uniform_residues(st["residues"], (count, 2), qs, n)
    top = min(qs) - 1
    e[:, ::3], e[:, 1::3] = top, -top
    out = ck.empty_u32((count, 2, limbs, n))
    ck.ckks_refresh(ctx, ck.to_device(ct), limbs, s_ntt, ck.to_device(a), ck.to_device(e), count, limbs, out)
    pick = sorted({0, count - 1})
    want = OR.refresh(ct[pick].astype(np.uint64), s, a[pick], e[pick], qs, psis, log_n, limbs).astype(np.uint32)
    assert np.array_equal(ck.to_host_u32(out)[pick], want)
