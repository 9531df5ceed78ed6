"""The launch shape of an evaluation follows an estimate of its time, and a
program set may be read with rows or without them by the number of cases: the
outputs of every case, and the fitness, are the same bits for every shape,
whichever sizes the set was evaluated at before."""
import numpy as np
import pytest

import oracle
import paper_1601_00221_amd as gp
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fset,F,P", [(synth.FULL, 16, 700), (synth.FULL, 41, 300), (synth.FULL, 1, 5),
                                      (synth.ARITH3, 8, 500)])
def test_every_shape_gives_the_same_bits(fset, F, P):
    import torch
    sizes = [40000, 300, 1025, 6000, 300, 40000]
    rng = synth.rng_for(90 + F + P)
    pop = synth.ptc2_population(rng, P, fset, F, 1, 60, 0.1)
    X = synth.uniform_cases(rng, F, max(sizes), -4, 4)
    y = synth.uniform_cases(rng, 1, max(sizes), -1, 1)[0]
    ps = gp.ProgSet.tree(pop.tok, pop.cst, pop.off, F)
    ref = oracle.tree_outputs(pop.tok, pop.cst, pop.off, X[:, :300])
    whole = None
    for N in sizes:
        print("shapes: F %d P %d N %d" % (F, P, N), flush=True)
        Xd, yd = torch.from_numpy(X[:, :N].copy()).cuda(), torch.from_numpy(y[:N].copy()).cuda()
        out, fit, one = (gp.out_tensor(k, P, N) for k in ("cases", "sum_abs", "sum_abs"))
        ps.eval(Xd, None, "cases", out)
        ps.eval(Xd, yd, "sum_abs", fit)
        gp.gp_eval_tree(pop.tok, pop.cst, pop.off, Xd, yd, "sum_abs", one)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        if whole is None:
            whole = got
        same = (got.view(np.int32) == whole[:, :N].view(np.int32)) | (np.isnan(got) & np.isnan(whole[:, :N]))
        assert same.all(), np.argwhere(~same)[:4]
        ok = (got[:, :300].view(np.int32) == ref.view(np.int32)) | (np.isnan(got[:, :300]) & np.isnan(ref))
        assert ok.all(), np.argwhere(~ok)[:4]
        assert torch.equal(one.view(torch.int32), fit.view(torch.int32))
        with np.errstate(all="ignore"):
            want = np.abs(got - y[:N]).astype(np.float64).sum(1).astype(np.float32)
        fine = np.isfinite(want)
        # binary64 sums in another order, rounded once to binary32
        assert np.allclose(fit.cpu().numpy()[fine], want[fine], rtol=2e-7, atol=0.0)
