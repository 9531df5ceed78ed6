"""A program set's evaluation captured into a graph: every replay gives the
bits of the eager evaluation, with eager work and synchronizations between the
replays."""
import pytest

import paper_1601_00221_amd as gp
import synth

pytestmark = pytest.mark.gpu


def _set(fset, F, P, N):
    import torch
    rng = synth.rng_for(31 + N)
    pop = synth.ptc2_population(rng, P, fset, F, 1, 60, 0.1)
    X = torch.from_numpy(synth.uniform_cases(rng, F, N, -4, 4)).cuda()
    return gp.ProgSet.tree(pop.tok, pop.cst, pop.off, F), X, X[0].clone(), [gp.out_tensor("mse", P, N) for _ in range(3)]


# one launch that finishes its fitness; a reduction; rows; features in LDS
@pytest.mark.parametrize("how", ["eval", "eval_noalloc"])
@pytest.mark.parametrize("fset,F,P,N", [(synth.ARITH3, 8, 300, 300), (synth.ARITH3, 8, 300, 40000),
                                        (synth.FULL, 8, 100, 40000), (synth.KDD_SET, 41, 300, 3000)])
def test_replays_equal_the_eager_evaluation(how, fset, F, P, N):
    import torch
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):     # (the set is uploaded on the stream that is captured)
        ps, X, y, (out, ref, other) = _set(fset, F, P, N)
    evaluate = getattr(ps, how)
    # the first evaluation over so many cases may upload a layout, the second sees that its upload has passed
    for _ in range(2):
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            evaluate(X, y, "mse", ref)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    print("capturing %s: F %d P %d N %d" % (how, F, P, N), flush=True)
    with torch.cuda.graph(g, stream=s):
        evaluate(X, y, "mse", out)
    for _ in range(4):
        out.fill_(-7)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int32), ref.view(torch.int32))
        with torch.cuda.stream(s):
            evaluate(X, y, "sum_abs", other)
        torch.cuda.synchronize()

