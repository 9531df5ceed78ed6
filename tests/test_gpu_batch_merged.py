"""Jobs of a batch that share form, dataset, fitness kind and registers and
are evaluated as one population: each job gets the bits of its own
evaluation, whichever of the sets are launched by themselves."""
import numpy as np
import pytest

import paper_1601_00221_amd as gp
import synth
from tests.gpu_util import dev, gpu_linear, gpu_tree

pytestmark = pytest.mark.gpu


def _spec(F):
    """(population, dataset, kind) of each job.  Trees with and without sin/cos/exp/log, one program alone, more
    programs than a block's waves; register programs with constants, without a constant array, and over fewer
    registers; jobs of one set apart from each other in the batch; kinds and datasets that form sets of their own."""
    rng = synth.rng_for(11)
    tree = lambda P, n, fs: synth.ptc2_population(rng, P, fs, F, 1, n, 0.2)   # noqa: E731
    lin = lambda P, n, regs, c: synth.linear_population(rng, P, 1, n, synth.BASIC, regs, F, n_const=c)   # noqa: E731
    return [(tree(60, 120, synth.FULL), 0, "mse"), (lin(50, 200, 8, 3), 0, "mse"), (tree(1, 9, synth.ARITH3), 0, "mse"),
            (lin(30, 100, 8, 0), 0, "mse"), (tree(90, 60, synth.KDD_SET), 0, "mse"), (lin(20, 80, 8, 1), 0, "mse"),
            (tree(40, 80, synth.FULL), 1, "hits"), (lin(25, 90, 4, 2), 0, "mse"), (tree(35, 80, synth.ARITH3), 1, "hits"),
            (lin(15, 60, 8, 2), 1, "class_err"), (tree(17, 40, synth.SHUTTLE_SET), 1, "class_err"),
            (tree(5, 30, synth.FULL), 0, "sum_abs")]


@pytest.mark.parametrize("limit,sizes", [("0", (1003, 259)), ("4e6", (1003, 259)), ("4e6", (30011, 1))])
def test_merged_jobs_get_the_bits_of_their_own_evaluation(monkeypatch, limit, sizes):
    import torch
    F = 9
    rng = synth.rng_for(12)
    data = [(synth.uniform_cases(rng, F, n, -4, 4), np.rint(synth.gaussian_noise(rng, n, 2.0)).astype(np.float32))
            for n in sizes]
    dd = [(dev(X), dev(y)) for X, y in data]
    spec = _spec(F)
    outs = [gp.out_tensor(kind, pop.n_prog, 0) for pop, _, kind in spec]
    jobs = [gp.make_job(pop, ds, kind, o) for (pop, ds, kind), o in zip(spec, outs)]
    jobs[3].lcst = jobs[3].lcst_off = None      # (programs without constants)
    ref = [(gpu_tree if hasattr(pop, "tok") else gpu_linear)(pop, *data[ds], kind) for pop, ds, kind in spec]
    monkeypatch.setenv("GP2D_MERGED_WORK", limit)
    print("merged batch: limit %s, %s cases" % (limit, sizes), flush=True)
    for _ in range(2):
        for o in outs:
            o.fill_(-7)
        gp.gp_eval_batch(dd, jobs)
        torch.cuda.synchronize()
        for k, o in enumerate(outs):
            got = o.cpu().numpy()
            assert np.array_equal(got.view(np.int32), ref[k].view(np.int32)), (k, spec[k][2])
