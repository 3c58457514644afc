"""Column workgroups of the matrix-core kernels in the shapes that large sets do not reach.

Waves that finish several target groups one after another: from 16 rows a column on a
wave keeps the twiddles of its current group in LDS words of its own, as doubles for a
group of Q limbs and as integer pairs for one of P limbs, and writes the next group's over
them. Waves take more than one group only in launches with a workgroup for every CU (smaller
ones share a tile's groups between workgroups), hence the batches here: at least 256
tiles, with 10 and 12 groups for the 4 wave pairs of a 64-column and the 8 waves of a
32-column workgroup, the last of them P groups.

Workgroups with fewer columns left than they have lanes for: blocks shorter than 32 words in
32-column workgroups (whose lanes past the end load the last column and store nothing),
shorter than 64 in 64-column ones, down to the 8 words of the smallest block.

Every plan here is one that the library accepts; a refusal fails the test. Expected values
come from the oracle, bit for bit.
"""
import numpy as np
import pytest

import oracle
from synth import ciphertext_batch, uniform_key, uniform_residues

from gpu_util import dev, empty, first_mismatch, host, kernel_launches

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("log_r", [4, 5])
@pytest.mark.parametrize("dnum,log_n,ell,batch", [(10, 8, 40, 26), (5, 8, 45, 52)])
def test_groups_in_turn_on_one_wave(dnum, log_n, ell, batch, log_r):
    import paper_2603_16692_amd as ks
    G, P = ks.KsParams(dnum, log_n, ell), oracle.Params(dnum, log_n, ell)
    d, evk = ciphertext_batch(P.q, P.n, batch), uniform_key(P.moduli, P.n, P.ndig)
    ref = oracle.keyswitch(P, d, evk, batch)
    plan = ks.make_plan(ks.DPOB, 1, log_r)
    out = empty(ref.shape)
    G.keyswitch(dev(d), dev(evk), out, batch, G.workspace(batch, plan), plan)
    mm = first_mismatch(host(out), ref)
    assert mm is None, f"{plan}: first mismatch {mm}"


# 32-column workgroups at 8 rows (6 steps of four sources and more), 16 (3 to 5) and 32 (3),
# 64-column ones below; digits that fill their last step and that leave 3 of 4 sources empty
@pytest.mark.parametrize("dnum,log_n,ell,log_r,columns", [
    (2, 8, 19, 5, 32), (2, 8, 20, 5, 32), (1, 8, 9, 5, 32), (2, 8, 19, 4, 32), (2, 7, 24, 4, 32), (1, 8, 17, 4, 32),
    (1, 7, 20, 4, 32), (2, 7, 50, 3, 32), (1, 6, 32, 3, 32), (2, 8, 42, 3, 32), (2, 8, 16, 5, 64), (2, 8, 8, 5, 64),
    (2, 7, 16, 4, 64), (2, 8, 8, 3, 64), (1, 6, 20, 3, 64), (1, 3, 32, 0, 64), (1, 5, 13, 2, 64)])
def test_fewer_columns_than_lanes(dnum, log_n, ell, log_r, columns):
    import paper_2603_16692_amd as ks
    G, P = ks.KsParams(dnum, log_n, ell), oracle.Params(dnum, log_n, ell)
    batch = 3
    d, evk = ciphertext_batch(P.q, P.n, batch), uniform_key(P.moduli, P.n, P.ndig)
    ref = oracle.keyswitch(P, d, evk, batch)
    dd, ee = dev(d), dev(evk)
    for plan in (ks.make_plan(ks.DPOB, 1, log_r), ks.make_plan(ks.DPOB, 1, log_r, hoist=True),
                 ks.make_plan(ks.DPOC, 3, log_r), ks.make_plan(ks.STAGED, 1, log_r)):
        out, ws = empty(ref.shape), G.workspace(batch, plan)
        cols = [k for k in kernel_launches(lambda s: G.keyswitch(dd, ee, out, batch, ws, plan, stream=s))
                if "_cols" in k.name]
        steps = -(-G.alpha // 4)
        assert cols and all(k.name.endswith("_cols_mx") and k.args[:2] == (log_r, steps) for k in cols)
        assert (32 if steps << log_r > (64 if log_r == 5 else 40) else 64) == columns
        mm = first_mismatch(host(out), ref)
        assert mm is None, f"{plan}: first mismatch {mm}"


# ks_bconv on the matrix cores takes 8 rows: N / 8 columns, 32 a workgroup from 6 steps on
@pytest.mark.parametrize("dnum,log_n,ell", [(1, 3, 32), (1, 5, 25), (1, 7, 21), (1, 7, 24), (1, 6, 17), (2, 4, 40)])
def test_bconv_with_fewer_columns_than_lanes(dnum, log_n, ell):
    import paper_2603_16692_amd as ks
    G, P = ks.KsParams(dnum, log_n, ell), oracle.Params(dnum, log_n, ell)
    batch = 2
    for j in (0, ks.KS_SET_P):
        mods = P.p if j < 0 else [P.moduli[i] for i in P.digit(j)]
        x = np.stack([uniform_residues(30 + b, mods, P.n) for b in range(batch)])
        ref = oracle.bconv(P, j, x, batch)
        xd, out = dev(x), empty(ref.shape)
        assert [k.name for k in kernel_launches(lambda s: G.bconv(xd, j, out, batch, stream=s))] == ["k_bconv_mx"]
        mm = first_mismatch(host(out), ref)
        assert mm is None, f"set {j}: first mismatch {mm}"


# The plans of the number-of-sources test that accept no refusal: all of these run, and the
# first split that stages more than 160 KB of digits is refused
@pytest.mark.parametrize("dnum,ell,log_r", [(2, 6, 5), (2, 8, 5), (2, 19, 5), (2, 24, 4), (1, 16, 4), (2, 33, 4),
                                            (2, 50, 3), (1, 32, 3), (1, 33, 3)])
def test_splits_accepted_and_refused(dnum, ell, log_r):
    import paper_2603_16692_amd as ks
    G = ks.KsParams(dnum, 13, ell)
    for df, chunks in ((ks.DPOB, 1), (ks.DSOC, 2), (ks.STAGED, 1)):
        assert G.workspace_bytes(2, ks.make_plan(df, chunks, log_r)) > 0
    first = next((r for r in range(log_r + 1, 6) if G.alpha << r > 320), 6)
    for r in range(6):
        plan = ks.make_plan(ks.DPOB, 1, r)
        if r < first:
            assert G.workspace_bytes(2, plan) > 0
        else:
            with pytest.raises(ks.KsError) as e:
                G.workspace_bytes(2, plan)
            assert e.value.code == ks.KS_EUNSUP
