"""Column workgroups whose waves finish several target groups one after another.

From 16 rows a column on a wave keeps the twiddles of its current group in LDS words
of its own, as doubles for a group of Q limbs and as integer pairs for one of P limbs,
and writes the next group's over them. Waves take more than one group only in launches
with a workgroup for every CU (smaller ones share a tile's groups between workgroups),
hence the batches here: at least 256 tiles, with 10 and 12 groups for the 4 wave pairs
of a 64-column and the 8 waves of a 32-column workgroup, the last of them P groups. Expected
values come from the oracle, bit for bit.
"""
import pytest

import oracle
from synth import ciphertext_batch, uniform_key

from gpu_util import dev, empty, first_mismatch, host

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
