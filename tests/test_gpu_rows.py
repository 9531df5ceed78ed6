"""Trees whose functions of a feature are read from rows that a block computes
once for its tile: outputs are the oracle's bits, for populations smaller and
larger than a block's waves, single and ragged tiles, and feature counts on
each kernel that has rows (among them one whose LDS holds only part of them);
and the fitness of every program equals the fitness of its outputs."""
import numpy as np
import pytest

import oracle
import paper_1601_00221_amd as gp
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,P,N", [(1, 9, 1), (3, 40, 257), (8, 300, 1023), (12, 60, 2048), (16, 260, 700),
                                   (24, 500, 300), (41, 33, 511), (41, 1500, 515)])
def test_rows_match_oracle(F, P, N):
    import torch
    rng = synth.rng_for(60 + F + P)
    pop = synth.ptc2_population(rng, P, synth.FULL, F, 1, 60, 0.1)
    X = synth.uniform_cases(rng, F, N, -4, 4)
    y = synth.uniform_cases(rng, 1, N, -1, 1)[0]
    Xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    ps = gp.ProgSet.tree(pop.tok, pop.cst, pop.off, F)
    out = gp.out_tensor("cases", P, N)
    fit = gp.out_tensor("sum_abs", P, N)
    print("rows: F %d P %d N %d" % (F, P, N), flush=True)
    for _ in range(2):
        ps.eval(Xd, None, "cases", out)
        ps.eval(Xd, yd, "sum_abs", fit)
    torch.cuda.synchronize()
    got, ref = out.cpu().numpy(), oracle.tree_outputs(pop.tok, pop.cst, pop.off, X)
    ok = (got.view(np.int32) == ref.view(np.int32)) | (np.isnan(got) & np.isnan(ref))
    assert ok.all(), np.argwhere(~ok)[:4]
    with np.errstate(all="ignore"):
        want = np.abs(got - y).astype(np.float64).sum(1).astype(np.float32)
    f = fit.cpu().numpy()
    fine = np.isfinite(want)
    # binary64 sums in another order, rounded once to binary32
    assert np.allclose(f[fine], want[fine], rtol=2e-7, atol=0.0)
    assert (np.isfinite(f) == fine).all()
