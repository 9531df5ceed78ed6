"""Every compiled kernel that can hold them gives the oracle's bits for trees
of its functions, forced for a program set, and the bits of the default kernel
where a batch of trees names it."""
import os
import sys

import numpy as np
import pytest

import oracle
import paper_1601_00221_amd as gp
import synth

sys.path.insert(0, os.path.join(os.path.dirname(gp.__file__), "csrc"))
import gen_core  # noqa: E402
sys.path.pop(0)

pytestmark = pytest.mark.gpu
# (from the generator: the library is not loaded while tests are collected, which may be before torch has loaded HIP)
BOOLEAN = [v[4] == 2 for v in gen_core.VARIANTS + gen_core.RING_VARIANTS]


def _same(a, b):
    return ((a.view(np.int32) == b.view(np.int32)) | (np.isnan(a) & np.isnan(b))).all()


@pytest.mark.parametrize("vi", [i for i, b in enumerate(BOOLEAN) if not b])
def test_kernel_on_trees(monkeypatch, vi):
    import torch
    v = gp.variants()[vi]
    F, N = min(8, v["n_feat"]), 512 * 3 + 77
    rng = synth.rng_for(70 + vi)
    pop = synth.ptc2_population(rng, 90, synth.SHUTTLE_SET if v["no_transc"] else synth.KDD_SET, F, 1, 24, 0.2)
    X = synth.uniform_cases(rng, F, N, -4, 4)
    y = synth.uniform_cases(rng, 1, N, -1, 1)[0]
    Xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    out, fit = gp.out_tensor("cases", pop.n_prog, N), gp.out_tensor("sum_abs", pop.n_prog, N)
    ref_fit = gp.out_tensor("sum_abs", pop.n_prog, N)
    monkeypatch.delenv("GP2D_VARIANT", raising=False)
    ps = gp.ProgSet.tree(pop.tok, pop.cst, pop.off, F)
    assert ps.info()["max_depth"] <= v["depth"]
    ps.eval(Xd, yd, "sum_abs", ref_fit)
    monkeypatch.setenv("GP2D_VARIANT", str(vi + 1))
    assert ps.info()["variant"] == vi
    print("kernel %s" % v["kernel"], flush=True)
    ps.eval(Xd, None, "cases", out)
    ps.eval(Xd, yd, "sum_abs", fit)
    torch.cuda.synchronize()
    assert _same(out.cpu().numpy(), oracle.tree_outputs(pop.tok, pop.cst, pop.off, X))
    assert _same(fit.cpu().numpy(), ref_fit.cpu().numpy())
    fit.fill_(-7)
    gp.gp_eval_batch([(Xd, yd)], [gp.make_job(pop, 0, "sum_abs", fit)], gp.BatchConfig(vi, 8, 1, 0))
    torch.cuda.synchronize()
    assert _same(fit.cpu().numpy(), ref_fit.cpu().numpy())


@pytest.mark.parametrize("vi", [i for i, b in enumerate(BOOLEAN) if b])
def test_kernel_on_boolean_trees(monkeypatch, vi):
    import torch
    v = gp.variants()[vi]
    F, N = 11, 32 * 700 + 5
    rng = synth.rng_for(170 + vi)
    pop = synth.ptc2_population(rng, 90, synth.BOOL_SET, F, 1, 40, 0.0)
    words = rng.integers(0, 1 << 32, (F + 1, (N + 31) // 32), dtype=np.uint32)
    Xd, yd = (torch.from_numpy(a.view(np.int32).copy()).cuda() for a in (words[:F], words[F]))
    hits, ref = (torch.empty(pop.n_prog, dtype=torch.int32, device="cuda") for _ in range(2))
    monkeypatch.delenv("GP2D_VARIANT", raising=False)
    ps = gp.ProgSet.boolean(pop.tok, pop.off, F)
    assert ps.info()["max_depth"] <= v["depth"]
    ps.eval(Xd, yd, "hits", ref, n_cases=N)
    monkeypatch.setenv("GP2D_VARIANT", str(vi + 1))
    assert ps.info()["variant"] == vi
    print("kernel %s" % v["kernel"], flush=True)
    ps.eval(Xd, yd, "hits", hits, n_cases=N)
    torch.cuda.synchronize()
    assert torch.equal(hits, ref)
