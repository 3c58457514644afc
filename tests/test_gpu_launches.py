"""Which kernels the library launches, where a rule on sizes chooses.

The rules choose between kernels that give the same words, so comparing results cannot
show that a call takes the wrong one; these tests read the launches of a captured call. Where
a line divides two kernels, the calls on both sides of it are compared with the
oracle bit for bit as well.
"""
import numpy as np
import pytest

import oracle
from synth import uniform_key, uniform_residues

from gpu_util import dev, empty, first_mismatch, host, kernel_launches

pytestmark = pytest.mark.gpu


# (dnum, log_n, ell, source set, batch): the products sources x targets x N x batch on either
# side of 5 * 2^19 from a digit (4 and 12 sources) and of 2^20 from P (4 and 6), and the
# numbers of sources just past those that have a line (16 and 8 below N = 2^8)
@pytest.mark.parametrize("dnum,log_n,ell,src,batch,kernel", [
    (1, 3, 4, 0, 1, "k_bconv"), (2, 13, 8, 0, 9, "k_bconv"), (2, 13, 8, 0, 11, "k_bconv_mx"),
    (2, 12, 24, 0, 2, "k_bconv"), (2, 12, 24, 0, 3, "k_bconv_mx"), (2, 8, 26, 1, 1, "k_bconv_mx"),
    (1, 6, 16, 0, 2, "k_bconv"), (1, 7, 17, 0, 1, "k_bconv_mx"),
    (2, 13, 8, -1, 4, "k_bconv"), (2, 13, 8, -1, 5, "k_bconv_mx"), (3, 12, 18, -1, 2, "k_bconv"),
    (3, 12, 18, -1, 3, "k_bconv_mx"), (1, 8, 7, -1, 1, "k_bconv_mx"), (1, 7, 8, -1, 2, "k_bconv"),
    (1, 6, 9, -1, 1, "k_bconv_mx"), (2, 13, 6, 0, 40, "k_bconv")])
def test_bconv_by_size(dnum, log_n, ell, src, batch, kernel):
    import paper_2603_16692_amd as ks
    G, P = ks.KsParams(dnum, log_n, ell), oracle.Params(dnum, log_n, ell)
    mods = P.p if src < 0 else [P.moduli[i] for i in P.digit(src)]
    x = np.stack([uniform_residues(90 + b, mods, P.n) for b in range(batch)])
    ref = oracle.bconv(P, src, x, batch)
    xd, out = dev(x), empty(ref.shape)
    launches = kernel_launches(lambda s: G.bconv(xd, src, out, batch, stream=s))
    assert [k.name for k in launches] == [kernel]
    mm = first_mismatch(host(out), ref)
    assert mm is None, f"first mismatch {mm}"


# below 3 * 2^18 coefficients (batch x limbs x N), and 2^22 of ext, one item and one coefficient a thread, else two
# coefficients, of two items where there are two; limbs shorter than a workgroup, a last odd
# item, more digits than a sum holds unfolded (9, 10)
@pytest.mark.parametrize("dnum,log_n,ell,batch,args", [
    (2, 3, 4, 5, (1, 1)), (9, 8, 9, 3, (1, 1)), (10, 10, 10, 1, (1, 1)), (2, 13, 10, 6, (1, 1)),
    (2, 16, 8, 1, (1, 2)), (2, 13, 8, 8, (2, 2)), (10, 13, 10, 9, (2, 2)),
    (10, 12, 10, 9, (1, 1)), (10, 12, 10, 10, (2, 2))])
def test_keymult_by_size(dnum, log_n, ell, batch, args):
    import paper_2603_16692_amd as ks
    G, P = ks.KsParams(dnum, log_n, ell), oracle.Params(dnum, log_n, ell)
    ext = np.stack([[uniform_residues(70 + b * P.ndig + j, P.moduli, P.n) for j in range(P.ndig)]
                    for b in range(batch)])
    top = np.array(P.moduli, dtype=np.uint64)[:, None] - np.uint64(1)
    ext[..., ::3] = top
    evk = uniform_key(P.moduli, P.n, P.ndig)
    evk[..., ::2] = top
    ref = oracle.keymult(P, ext, evk, batch)
    xd, kd, acc = dev(ext), dev(evk), empty(ref.shape)
    launches = kernel_launches(lambda s: G.keymult(xd, kd, acc, batch, stream=s))
    assert [(k.name, k.args) for k in launches] == [("k_keymult", args)]
    mm = first_mismatch(host(acc), ref)
    assert mm is None, f"first mismatch {mm}"


# blocks of 2^14 run 16 elements on each of 1024 threads, which have 128 registers: what
# KeyMult loads ahead of use beyond them only goes to scratch memory and back (bytes a lane)
@pytest.mark.parametrize("dataflow", ["DPOB", "DSOB"])
def test_keymult_scratch_memory_at_the_largest_blocks(dataflow):
    import paper_2603_16692_amd as ks
    G = ks.KsParams(2, 14, 4)
    plan = ks.make_plan(getattr(ks, dataflow), 1, 0)
    sh = G.shapes(1)
    d, evk, out, ws = empty(sh["d"]).zero_(), empty(sh["evk"]).zero_(), empty(sh["out"]), G.workspace(1, plan)
    found = [k for k in kernel_launches(lambda s: G.keyswitch(d, evk, out, 1, ws, plan, stream=s))
             if k.name == "k_keymult_blocks"]
    assert found and all(k.args[:2] == (14, 4) for k in found)
    assert all(k.scratch <= 128 for k in found), found


# the column kernels with 32 rows keep everything in registers (1, 2, 3 steps of four
# sources: 64 columns and 32)
@pytest.mark.parametrize("ell", [8, 16, 20])
def test_column_kernels_of_32_rows_use_no_scratch_memory(ell):
    import paper_2603_16692_amd as ks
    G = ks.KsParams(2, 8, ell)
    plan = ks.make_plan(ks.DPOB, 1, 5)
    sh = G.shapes(1)
    d, evk, out, ws = empty(sh["d"]).zero_(), empty(sh["evk"]).zero_(), empty(sh["out"]), G.workspace(1, plan)
    found = [k for k in kernel_launches(lambda s: G.keyswitch(d, evk, out, 1, ws, plan, stream=s))
             if k.name in ("k_modup_cols_mx", "k_moddown_cols_mx")]
    assert [k.args[:2] for k in found] == [(5, -(-ell // 8))] * 2
    assert not any(k.scratch for k in found), found


# the tuner leaves out the plan with the matrix-core flag where distinct_plans says that it
# launches what the plan without it does
@pytest.mark.parametrize("dnum,log_n,ell,level", [(2, 9, 8, 8), (2, 9, 6, 6), (1, 9, 16, 16), (2, 9, 16, 4),
                                                  (2, 9, 16, 3)])
def test_flag_twins_launch_the_same_kernels(dnum, log_n, ell, level):
    import paper_2603_16692_amd as ks
    from paper_2603_16692_amd import autotune
    top = ks.KsParams(dnum, log_n, ell)
    G = top if level == ell else top.at_level(level)
    d, evk, out = empty(G.shapes(2)["d"]).zero_(), empty(top.shapes(1)["evk"]).zero_(), empty(G.shapes(2)["out"])

    def launches(plan):
        ws = G.workspace(2, plan)
        return kernel_launches(lambda s: G.keyswitch(d, evk, out, 2, ws, plan, stream=s))

    plans = [p for p in autotune.candidate_plans(G, 2, chunk_range=(2,)) if p.flags & ks.PLAN_MFMA_BCONV]
    kept = {p.key() for p in autotune.distinct_plans(G, autotune.candidate_plans(G, 2, chunk_range=(2,)))}
    assert plans
    for p in plans:
        twin = ks.Plan(p.dataflow, p.chunks, p.log_r, p.flags & ~ks.PLAN_MFMA_BCONV, p.batch_tile)
        assert (launches(p) == launches(twin)) == (p.key() not in kept), p
