"""Scenarios of the library's host runtime, on a HIP runtime of host memory
(fake_hip.cpp).

    python host_scenarios.py LIBGP SCENARIO [ARGUMENT ...]

Started by tests/test_host_runtime.py, one process a scenario; the last line
is "ok" if every check held."""
import ctypes as C
import os
import sys

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
sys.path.insert(0, ROOT)

import paper_1601_00221_amd as gp  # noqa: E402
import synth                       # noqa: E402

gp.LIB_PATH = sys.argv[1]
gp.stream_ptr = lambda stream=None: None   # the null stream
LAUNCHES, ROWS, GROUPS, VARIANT, TABLE, BAD_LAYOUTS, UPLOADS, LOWERED = range(8)


def fake(what):
    return gp.lib().fake_int(what)


class Array:
    """Stands for a device tensor: a numpy array the fake runtime takes as device memory."""

    def __init__(self, a):
        self.a, self.shape = np.ascontiguousarray(a), a.shape

    def data_ptr(self):
        return self.a.ctypes.data


def tree_set(rng, P, F, fset):
    pop = synth.ptc2_population(rng, P, fset, F, 1, 60, 0.1)
    return gp.ProgSet.tree(pop.tok, pop.cst, pop.off, F)


def evaluate(ps, X, y, out, N):
    gp.check(gp.lib().gp_progset_eval(ps._h, X.data_ptr(), X.shape[0], N, y.data_ptr(), gp.kind_id("sum_abs"),
                                      out.data_ptr(), None))


def failed_allocation_leaves_no_layout():
    """An evaluation whose k-th allocation fails reports it and launches nothing; the next one uploads what is missing
    and launches with a whole layout."""
    rng = synth.rng_for(5)
    F, P, N = 16, 700, 3000
    X, y, out = Array(np.zeros((F, N), np.float32)), Array(np.zeros(N, np.float32)), Array(np.zeros(P, np.float32))
    failures = 0
    for _ in range(4):
        tree_set(rng, P, F, synth.FULL).close()   # (the staging buffers are there)
    for k in range(1, 12):
        ps = tree_set(rng, P, F, synth.FULL)
        launched = fake(LAUNCHES)
        gp.lib().fake_fail_malloc(k)
        try:
            evaluate(ps, X, y, out, N)
            assert fake(LAUNCHES) == launched + 1
        except gp.GPError as e:
            assert e.status == -2, e
            assert fake(LAUNCHES) == launched
            failures += 1
        gp.lib().fake_fail_malloc(0)
        for _ in range(6):
            evaluate(ps, X, y, out, N)
            assert fake(BAD_LAYOUTS) == 0, (k, fake(BAD_LAYOUTS))
        ps.close()
    assert failures > 0


def batch(rng, specs, F, N):
    """A dataset and jobs: (trees?, programs, length)."""
    X, y = Array(np.zeros((F, N), np.float32)), Array(np.zeros(N, np.float32))
    jobs = []
    for tree, P, n in specs:
        pop = synth.ptc2_population(rng, P, synth.FULL, F, 1, n, 0.1) if tree else \
            synth.linear_population(rng, P, 1, n, synth.BASIC, 8, F, n_const=2)
        jobs.append(gp.make_job(pop, 0, "mse", 0x10000))
    return [(X, y)], jobs


def batch_is_lowered_once():
    """gp_eval_batch without a configuration lowers every program once, merged sets and the others."""
    for limit, launches in (("0", 2), ("1e18", 1)):
        os.environ["GP2D_MERGED_WORK"] = limit
        data, jobs = batch(synth.rng_for(6), [(True, 70, 40), (False, 50, 60), (True, 30, 40)], 8, 1000)
        lowered, launched = fake(LOWERED), fake(LAUNCHES)
        gp.gp_eval_batch(data, jobs)
        assert fake(LAUNCHES) - launched == launches
        assert fake(LOWERED) - lowered == 150, fake(LOWERED) - lowered


def every_evaluation_takes_the_translation_that_suits_it():
    """A small set of trees with sin/cos/exp/log is uploaded with rows and without when it is created: every evaluation
    takes the translation that suits its number of cases, the first as the later ones, and the first over a number of
    cases uploads its layout alone, the later ones nothing.  Where there was no memory for both, the rows serve; a
    large set, whose rows always pay, is uploaded with them alone."""
    rng = synth.rng_for(5)
    F, P, few, many = 8, 700, 300, 1000000
    X, y, out = Array(np.zeros((F, many), np.float32)), Array(np.zeros(many, np.float32)), Array(np.zeros(P, np.float32))
    for _ in range(4):
        tree_set(rng, P, F, synth.FULL).close()   # (the kernel is set up and the staging buffers are there)
    for k in range(1, 8):
        gp.lib().fake_fail_malloc(0 if k == 7 else k)
        try:
            ps = tree_set(rng, P, F, synth.FULL)
        except gp.GPError as e:
            assert e.status == -2, e
            continue
        finally:
            gp.lib().fake_fail_malloc(0)
        rows = []
        for n in (few, few, many, few, many):
            uploads = fake(UPLOADS)
            evaluate(ps, X, y, out, n)
            rows.append(fake(ROWS))
            assert fake(UPLOADS) - uploads <= (len(rows) == 1), (k, rows)
        assert rows[2] > 0 and rows[2] == rows[4] and rows[0] == rows[1] == rows[3]
        assert rows[0] == 0 or k < 7, (k, rows)
        assert fake(BAD_LAYOUTS) == 0
        ps.close()
    pop = synth.ptc2_population(rng, 1000, synth.FULL, F, 1, 250, 0.1)
    uploads = fake(UPLOADS)
    ps = gp.ProgSet.tree(pop.tok, pop.cst, pop.off, F)
    assert fake(UPLOADS) - uploads == 2       # code and layout
    evaluate(ps, X, y, Array(np.zeros(1000, np.float32)), few)
    assert fake(ROWS) > 0


MIXED = [(True, 70, 40), (False, 50, 60)]


def tune():
    """Tunes a batch; prints the kernel and its number."""
    os.environ["GP2D_MERGED_WORK"] = "1e18"
    gp.lib().fake_times(C.c_double(5.0), C.c_double(1.0), C.c_double(0.0))
    best, _ = gp.gp_tune_batch(*batch(synth.rng_for(7), MIXED, 8, 1000))
    print(gp.variants()[best.variant]["kernel"], best.variant, flush=True)


def evaluated_with(kernel):
    """The same batch without a configuration is evaluated, by the kernel named (or any: "-")."""
    os.environ["GP2D_MERGED_WORK"] = "1e18"
    launched = fake(LAUNCHES)
    gp.gp_eval_batch(*batch(synth.rng_for(7), MIXED, 8, 1000))
    assert fake(LAUNCHES) == launched + 1 and fake(TABLE) == 1
    name = gp.variants()[fake(VARIANT)]["kernel"]
    print(name, flush=True)
    assert kernel in ("-", name), name


def tuning_keeps_the_faster(launch, table, copy, table_kept):
    """A batch of two sets is tuned; evaluations then take the table of units, or the sets' own launches, whichever
    whole call is the shorter: 5 copies and a launch of `table` ms, or 4 copies and two launches of `launch` ms."""
    os.environ["GP2D_MERGED_WORK"] = "0"
    gp.lib().fake_times(*(C.c_double(float(t)) for t in (launch, table, copy)))
    data, jobs = batch(synth.rng_for(7), MIXED, 8, 1000)
    _, ms = gp.gp_tune_batch(data, jobs)
    assert abs(ms - float(table)) < 1e-3, ms
    uploads = fake(UPLOADS)
    gp.gp_eval_batch(data, jobs)
    assert fake(TABLE) == int(table_kept)
    assert fake(UPLOADS) - uploads == (5 if int(table_kept) else 4)


def tuning_does_without_the_default():
    """Where the default launches cannot be made (no memory), the tuned configuration is stored and returned."""
    gp.lib().fake_times(*(C.c_double(t) for t in (5.0, 1.0, 0.0)))
    data, jobs = batch(synth.rng_for(7), MIXED, 8, 1000)
    os.environ["GP2D_MERGED_WORK"] = "1e18"
    gp.gp_tune_batch(data, jobs)              # (the table route's buffers are there)
    os.environ["GP2D_MERGED_WORK"] = "0"
    gp.lib().fake_fail_malloc(1)
    gp.gp_tune_batch(data, jobs)
    gp.lib().fake_fail_malloc(0)
    gp.gp_eval_batch(data, jobs)
    assert fake(TABLE) == 1


SCENARIOS = {f.__name__: f for f in (failed_allocation_leaves_no_layout, batch_is_lowered_once, tune, evaluated_with,
                                     tuning_keeps_the_faster, tuning_does_without_the_default,
                                     every_evaluation_takes_the_translation_that_suits_it)}

if __name__ == "__main__":
    SCENARIOS[sys.argv[2]](*sys.argv[3:])
    print("ok", flush=True)
