"""gp_core_lower_tree with features beyond a kernel's slots: kernels that hold
features in registers alone give one instruction per lowered instruction,
whatever the feature; the kernel that holds others in LDS pushes those up to
its limit, and refuses more."""
import os
import sys

import numpy as np
import pytest

import paper_1601_00221_amd as gp
import synth

sys.path.insert(0, os.path.join(os.path.dirname(gp.__file__), "csrc"))
import gen_core  # noqa: E402
sys.path.pop(0)

BASE = 0x7F0000000000
# (from the generator: the library is not loaded while tests are collected, which may be before torch has loaded HIP)
VARIANTS = [i for i, v in enumerate(gen_core.VARIANTS + gen_core.RING_VARIANTS) if v[4] != 2]


class _Tree:
    def __init__(self, tok):
        self.tok, self.cst = np.array(tok, np.int32), np.zeros(len(tok), np.float32)
        self.off, self.n_prog = np.array([0, len(tok)], np.int64), 1


def _var(f):
    return synth.VAR | (f << 8)


# tree, its core instructions with the end, and those where every feature named is pushed first
TREES = [(lambda f: [synth.SIN, _var(f)], 2, 3), (lambda f: [synth.PLOG, _var(f)], 2, 3), (lambda f: [_var(f)], 2, 2),
         (lambda f: [synth.ADD, _var(f), _var(f)], 2, 4), (lambda f: [synth.PDIV, _var(f), synth.CONST], 2, 3),
         (lambda f: [synth.GT, _var(0), _var(f)], 2, 3)]


@pytest.mark.parametrize("vi", VARIANTS)
def test_features_beyond_the_slots(vi):
    v = gp.variants()[vi]
    wide = v["kernel"] == "k_core_4_9_11_48_t"
    for f in sorted({0, v["n_feat"] - 1, v["n_feat"], v["n_feat"] + 1, 43, 44, 100, 249, 254}):
        for tree, plain, pushed in TREES:
            if wide and f >= 44:
                with pytest.raises(gp.GPError, match="takes 44 features"):
                    gp.core_lower(_Tree(tree(f)), 255, vi, BASE)
                continue
            words, prog_off = gp.core_lower(_Tree(tree(f)), 255, vi, BASE)
            lds = wide and f >= v["n_feat"]
            assert prog_off[0] == 0
            payload = words.reshape(-1, 4)[:, 2]
            end = int(np.flatnonzero(payload >> 24 == 15)[0])
            assert end + 1 == (pushed if lds else plain), (v["kernel"], f, end)
