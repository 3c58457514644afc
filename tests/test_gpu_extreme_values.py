"""KeySwitch on residues at the ends of their range.

Between the passes the kernels hold values well outside [0, modulus) (lazy sums
within 8q of a Q prime, below 2^64 for a P prime) and make canonical residues
only at the boundary and before a base conversion. Random residues rarely reach the
largest sums or the exact multiples of a modulus; the patterns here do: zeros,
q - 1 everywhere, alternating ends, a single one, half the modulus. Expected
values come from the oracle, bit for bit.
"""
import numpy as np
import pytest
import torch

import oracle

from gpu_util import dev, empty, first_mismatch, host

pytestmark = pytest.mark.gpu


def _pattern(name, moduli, n):
    x = np.zeros((len(moduli), n), dtype=np.uint64)
    top = np.array(moduli, dtype=np.uint64)[:, None] - np.uint64(1)
    if name == "top":
        x[:] = top
    elif name == "ends":
        x[:, 1::2] = top
    elif name == "one":
        x[:, n // 3] = 1
    elif name == "half":
        x[:] = top // np.uint64(2)
        x[:, ::3] += np.uint64(1)
    return x


# every first-round size and elements-per-thread count of the block passes:
# blocks of 2^8 to 2^14, remainders 1 to 4 of the stages over the rounds
@pytest.mark.parametrize("dnum,log_n,ell,log_rs", [(3, 12, 7, (0, 1, 2, 4)), (2, 14, 5, (0, 1, 3, 5)),
                                                   (5, 13, 10, (0, 3, 5)), (1, 9, 3, (0, 2)),
                                                   (11, 10, 11, (0, 2))])  # more digits than a sum holds unfolded
@pytest.mark.parametrize("pattern", ["top", "ends", "one", "half"])
def test_keyswitch_on_extreme_residues(dnum, log_n, ell, log_rs, pattern):
    import paper_2603_16692_amd as ks
    G, P = ks.KsParams(dnum, log_n, ell), oracle.Params(dnum, log_n, ell)
    batch = 2
    d = np.stack([_pattern(pattern, P.q, P.n), _pattern("top", P.q, P.n)])
    evk = np.stack([[_pattern("top", P.moduli, P.n), _pattern(pattern, P.moduli, P.n)] for _ in range(P.ndig)])
    ref = oracle.keyswitch(P, d, evk, batch)
    dd, ee = dev(d), dev(evk)
    for log_r in log_rs:
        for plan in (ks.make_plan(ks.DPOB, 1, log_r), ks.make_plan(ks.DPOB, 1, log_r, mfma=True),
                     ks.make_plan(ks.DPOB, 1, log_r, hoist=True), ks.make_plan(ks.DSOB, 1, log_r),
                     ks.make_plan(ks.STAGED, 1, log_r)):
            out = empty(ref.shape)
            G.keyswitch(dd, ee, out, batch, G.workspace(batch, plan), plan)
            mm = first_mismatch(host(out), ref)
            assert mm is None, f"{pattern} {plan}: first mismatch {mm}"


@pytest.mark.parametrize("log_n", [3, 6, 9, 11, 13, 14, 16])
@pytest.mark.parametrize("pattern", ["top", "ends", "one", "half"])
def test_transforms_of_extreme_residues(log_n, pattern):
    import paper_2603_16692_amd as ks
    G, P = ks.KsParams(2, log_n, 3), oracle.Params(2, log_n, 3)
    x = _pattern(pattern, P.moduli, P.n)
    for call, ref in ((G.ntt, oracle.ntt), (G.intt, oracle.intt)):
        want = np.stack([ref(P.moduli[t], P.psi[t], log_n, x[t]) for t in range(P.nl)])
        y = dev(x[None])
        call(y, 0, P.nl, 1)
        mm = first_mismatch(host(y)[0], want)
        assert mm is None, f"{call.__name__} {pattern}: first mismatch {mm}"
    torch.cuda.synchronize()
