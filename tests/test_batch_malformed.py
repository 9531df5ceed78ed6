"""gp_eval_batch on malformed program arrays: each call returns an error that
names the job, and reads nothing that the arrays do not hold.  (Every call in
a process of its own: reading past an array would end it.)"""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CALL = """
import ctypes as C, sys
import numpy as np
sys.path.insert(0, %r)
import paper_1601_00221_amd as gp
tree, off, coff, n_cases = eval(sys.argv[1])
keep = [np.array(a, dt) for a, dt in (([64], np.int32), ([0.0], np.float32), (off, np.int64),
                                      ([0], np.uint32), ([1.0], np.float32), (coff, np.int64))]
tok, tcst, offs, code, lcst, lcst_off = (a.ctypes.data for a in keep)
j = gp.Job()
j.form, j.n_prog, j.dataset, j.kind, j.out = (0 if tree else 1), len(off) - 1, 0, 1, 0x10000
if tree:
    j.tok, j.tcst, j.toff = tok, tcst, offs
else:
    j.code, j.loff, j.lcst, j.lcst_off, j.n_reg = code, offs, lcst, lcst_off, 8
d = gp.Dataset(0x10000, 2, n_cases, 0x10000)
rc = gp.lib().gp_eval_batch(C.byref(d), 1, C.byref(j), 1, None, None)
print(rc, gp.last_error())
""" % ROOT


@pytest.mark.parametrize("tree,off,coff,status,message", [
    (True, [0, 1 << 50], [0, 0], -3, "job 0: program 0: 1125899906842624 nodes exceeds 65536"),
    (True, [0, 40000000], [0, 0], -3, "job 0: program 0: 40000000 nodes exceeds 65536"),
    (True, [0, 1, 1 << 40], [0, 0, 0], -3, "job 0: program 1: 1099511627775 nodes exceeds 65536"),
    (True, [0, 1 << 40, 1], [0, 0, 0], -3, "job 0: program 0: 1099511627776 nodes exceeds 65536"),
    (True, [1, 1 << 40], [0, 0], -1, "job 0: off[0] must be 0"),
    (True, [0, 1, 1], [0, 0, 0], -1, "job 0: program 1 is empty"),
    (False, [0, 1 << 50], [0, 0], -3, "job 0: program 0: 1125899906842624 instructions exceeds 65536"),
    (False, [0, 1], [0, 1 << 40], -1, "job 0: program 0: 1099511627776 constants"),
    (False, [0, 1], [0, 129], -1, "job 0: program 0: 129 constants"),
    (False, [0, 1], [1, 2], -1, "job 0: cst_off[0] must be 0"),
])
def test_malformed_arrays_are_refused(tree, off, coff, status, message):
    for n_cases in (1000, 2000000000):   # a small set of jobs, and one that would be launched by itself
        r = subprocess.run([sys.executable, "-c", CALL, repr((tree, off, coff, n_cases))], capture_output=True,
                           text=True, timeout=120)
        assert r.returncode == 0, (r.returncode, r.stderr[-500:])
        assert r.stdout.strip() == "%d %s" % (status, message), r.stdout


@pytest.mark.parametrize("variant,status,message", [(4000, -1, "kernel variant 4000 does not exist"),
                                                    (1 << 30, -1, "kernel variant 1073741824 does not exist"),
                                                    (-1, -3, "no kernel variant can hold these programs"),
                                                    (22, -1, "variant 22 is a Boolean kernel")])
def test_unknown_kernels_are_refused(variant, status, message):
    call = CALL.replace("1, None, None)", "1, C.byref(gp.BatchConfig(%d, 8, 1, 0)), None)" % variant)
    r = subprocess.run([sys.executable, "-c", call, repr((True, [0, 1], [0, 0], 1000))], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, (r.returncode, r.stderr[-500:])
    assert r.stdout.strip() == "%d %s" % (status, message), r.stdout
