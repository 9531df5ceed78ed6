"""Evaluating a program set on one stream while another thread captures a graph
on another stream, in the default (global) capture mode: the evaluation asks
nothing that such a capture forbids, so both succeed, and the results are those
of an evaluation without the capture."""
import threading

import pytest

import paper_1601_00221_amd as gp
import synth

pytestmark = pytest.mark.gpu


def test_evaluation_beside_a_capture_on_another_stream():
    import torch
    # (cases enough for the layout that a set uploads when it is created: nothing is allocated by the evaluation)
    F, P, N = 8, 400, 4000000
    rng = synth.rng_for(3)
    pops = [synth.ptc2_population(rng, P, synth.ARITH3, F, 1, 60, 0.1) for _ in range(2)]
    X = torch.from_numpy(synth.uniform_cases(rng, F, N, -4, 4)).cuda()
    y = X[0].clone()
    stream = torch.cuda.Stream()
    out, ref = gp.out_tensor("sum_abs", P, N), gp.out_tensor("sum_abs", P, N)
    a = torch.ones(1000, device="cuda")
    side = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        first = gp.ProgSet.tree(pops[0].tok, pops[0].cst, pops[0].off, F)
        first.eval(X, y, "sum_abs", out)          # the stream's workspace and the kernel's first use
        second = gp.ProgSet.tree(pops[1].tok, pops[1].cst, pops[1].off, F)
    torch.cuda.synchronize()
    capturing, evaluated = threading.Event(), threading.Event()
    result = {}

    def capture():
        try:
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.stream(side):
                graph.capture_begin(capture_error_mode="global")
                try:
                    b = a + 1
                    capturing.set()
                    evaluated.wait(60)
                    c = b * 2
                finally:
                    graph.capture_end()
            graph.replay()
            torch.cuda.synchronize()
            result["sum"] = float(c.sum())
        except Exception as e:   # reported after the join
            result["error"] = repr(e)
            capturing.set()

    th = threading.Thread(target=capture)
    th.start()
    try:
        assert capturing.wait(60)
        print("evaluating beside a capture", flush=True)
        with torch.cuda.stream(stream):
            second.eval(X, y, "sum_abs", out)
    finally:
        evaluated.set()
        th.join()
    assert "error" not in result, result["error"]
    assert result["sum"] == 4000.0
    with torch.cuda.stream(stream):
        second.eval(X, y, "sum_abs", ref)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int32), ref.view(torch.int32))
