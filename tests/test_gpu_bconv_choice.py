"""The base conversion a plan without KS_PLAN_MFMA_BCONV picks by itself.

The column kernels choose between scalar products and the int8 matrix form by the
number of source primes, and the matrix form between 64 and 32 columns a workgroup
by the rows and sources its digits take in LDS. Digit sizes here lie on both sides of
each of those lines (3 / 4 sources, 16 / 17, 32 / 33; 2, 3 and 5 to 8 steps of
four at 8 to 32 rows), with short last digits and levels below a digit, against
the oracle bit for bit.
"""
import numpy as np
import pytest

import oracle
from synth import ciphertext_batch, uniform_key, uniform_residues

from gpu_util import dev, empty, first_mismatch, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dnum,log_n,ell,log_rs", [
    (2, 9, 6, (0, 2, 5)), (2, 9, 8, (0, 2, 5)), (2, 10, 19, (1, 3, 5)), (2, 10, 24, (3, 4)), (1, 10, 16, (3, 4)),
    (2, 10, 33, (0, 2, 3, 4)), (2, 13, 50, (2, 3)), (1, 9, 32, (2, 3)), (1, 9, 33, (2, 3))])
def test_keyswitch_by_number_of_sources(dnum, log_n, ell, log_rs):
    import paper_2603_16692_amd as ks
    G, P = ks.KsParams(dnum, log_n, ell), oracle.Params(dnum, log_n, ell)
    batch = 2
    d, evk = ciphertext_batch(P.q, P.n, batch), uniform_key(P.moduli, P.n, P.ndig)
    ref = oracle.keyswitch(P, d, evk, batch)
    dd, ee = dev(d), dev(evk)
    tried = 0
    for log_r in log_rs:
        for plan in (ks.make_plan(ks.DPOB, 1, log_r), ks.make_plan(ks.DSOC, 2, log_r),
                     ks.make_plan(ks.STAGED, 1, log_r)):
            try:
                ws = G.workspace(batch, plan)
            except ks.KsError as e:  # more digits than the scalar form's LDS takes: refused as before
                assert e.code == ks.KS_EUNSUP
                continue
            out = empty(ref.shape)
            G.keyswitch(dd, ee, out, batch, ws, plan)
            mm = first_mismatch(host(out), ref)
            assert mm is None, f"{plan}: first mismatch {mm}"
            tried += 1
    assert tried


@pytest.mark.parametrize("level", [1, 3, 5, 9, 12])
def test_levels_below_and_across_a_digit(level):
    import paper_2603_16692_amd as ks
    top, P = ks.KsParams(2, 10, 16), oracle.Params(2, 10, 16)
    G = top.at_level(level)
    d, evk = ciphertext_batch(P.q[:level], P.n, 1), uniform_key(P.moduli, P.n, P.ndig)
    ref = oracle.keyswitch(P.at_level(level), d, evk, 1)
    for log_r in (0, 3, 4):
        plan = ks.make_plan(ks.DPOB, 1, log_r)
        out = empty(ref.shape)
        G.keyswitch(dev(d), dev(evk), out, 1, G.workspace(1, plan), plan)
        mm = first_mismatch(host(out), ref)
        assert mm is None, f"level {level} {plan}: first mismatch {mm}"


@pytest.mark.parametrize("dnum,log_n,ell,batch", [
    (1, 3, 4, 2), (2, 9, 8, 3), (2, 10, 33, 1), (1, 11, 32, 1), (1, 9, 33, 1), (3, 12, 13, 5)])
def test_bconv_by_number_of_sources(dnum, log_n, ell, batch):
    import paper_2603_16692_amd as ks
    G, P = ks.KsParams(dnum, log_n, ell), oracle.Params(dnum, log_n, ell)
    for j in list(range(P.ndig)) + [ks.KS_SET_P]:
        mods = P.p if j < 0 else [P.moduli[i] for i in P.digit(j)]
        x = np.stack([uniform_residues(50 + b + 7 * j, mods, P.n) for b in range(batch)])
        x[0, :, ::5] = 0
        x[0, :, 1::5] = np.array(mods, dtype=np.uint64)[:, None] - np.uint64(1)
        ref = oracle.bconv(P, j, x, batch)
        out = empty(ref.shape)
        G.bconv(dev(x), j, out, batch)
        mm = first_mismatch(host(out), ref)
        assert mm is None, f"set {j}: first mismatch {mm}"


# one item and two a thread, a last odd item, limbs shorter than a workgroup's
# 512 elements, more digits than a sum holds unfolded
@pytest.mark.parametrize("dnum,log_n,ell,batch", [(2, 3, 4, 3), (3, 8, 5, 1), (11, 9, 11, 2), (9, 10, 9, 5)])
def test_keymult_shapes(dnum, log_n, ell, batch):
    import paper_2603_16692_amd as ks
    G, P = ks.KsParams(dnum, log_n, ell), oracle.Params(dnum, log_n, ell)
    ext = np.stack([[uniform_residues(70 + b * P.ndig + j, P.moduli, P.n) for j in range(P.ndig)]
                    for b in range(batch)])
    top = np.array(P.moduli, dtype=np.uint64)[:, None] - np.uint64(1)
    ext[..., ::3] = top
    evk = uniform_key(P.moduli, P.n, P.ndig)
    evk[..., ::2] = top
    ref = oracle.keymult(P, ext, evk, batch)
    acc = empty(ref.shape)
    G.keymult(dev(ext), dev(evk), acc, batch)
    mm = first_mismatch(host(acc), ref)
    assert mm is None, f"first mismatch {mm}"
