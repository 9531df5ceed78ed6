"""The whole interpreter block, executed on the CPU.

test_core_emulation runs the handlers; here the block they sit in runs too:
the load of a unit's tile, the code lines fetched ahead, the end of every
program with its fitness terms and their sum over the wave, the ragged last
tile, and sin/cos/exp/log.  The emulator executes the generated text, lane by
lane, with every memory access checked against the buffers it may touch, and
the partial sums (or outputs) must be the definition's bits: binary32 error
terms of the oracle's outputs, summed in binary64 over the four slots of a
block and then over the lanes 32, 16, 8, 4, 2 and 1 apart."""
import os
import re
import sys

import numpy as np
import pytest

import oracle
import paper_1601_00221_amd as gp
import synth

CSRC = os.path.join(os.path.dirname(gp.__file__), "csrc")
sys.path.insert(0, CSRC)
import gen_core  # noqa: E402

sys.path.pop(0)

ALL = gen_core.VARIANTS + gen_core.RING_VARIANTS
CODE, XBASE, YBASE, PART, CASES, COEF = (0x100000000 * k for k in (16, 32, 48, 64, 80, 96))
TEXT = 0x7F0000000000
M32, M64 = 0xFFFFFFFF, 0xFFFFFFFFFFFFFFFF
LANES = np.arange(64)


def tables():
    """The block's LDS tables and coefficients, from the generated header and their definitions."""
    text = open(os.path.join(CSRC, "gp_math_tables.h")).read()

    def arr(name):
        body = re.search(name + r"\[\d+\] = \{([^}]*)\}", text).group(1)
        return [float.fromhex(x.strip()) for x in body.split(",") if x.strip()]
    tab = np.array(arr("kSinCos") + arr("kExp2J") + arr("kLogCT") + arr("kPiChunks"))
    h = float.fromhex
    co = [h("0x1.45f306dc9c883p+4"), h("0x1.921fb54442d18p-5"), h("0x1.1a62633145c07p-59"),
          -h("0x1.f1976b7ed8fbcp-115"), -1 / 6, -1 / 5040, -1 / 720, h("0x1.71547652b82fep+6"),
          h("0x1.62e42fefa39efp-7"), h("0x1.abc9e3b39803fp-62"), 1 / 6, 1 / 120, h("0x1.62e42fefa39efp-1"),
          1 / 3, -0.25, -1 / 6]
    return tab, np.array(co)


def fma(a, b, c):
    """a b + c of binary64 arrays: the product and the sum with their exact errors, which are then added (one
    rounding but for rare ties); plain arithmetic where that overflows or is not finite."""
    split = lambda t: (t * 134217729.0) - ((t * 134217729.0) - t)   # noqa: E731
    p = a * b
    ah, bh = split(a), split(b)
    al, bl = a - ah, b - bh
    ep = ((ah * bh - p) + ah * bl + al * bh) + al * bl
    s = p + c
    bb = s - p
    es = (p - (s - bb)) + (c - bb)
    r = s + (es + ep)
    return np.where(np.isfinite(r) & (s != 0), r, np.where(np.isfinite(ep) & (s == 0) & (ep != 0), ep, s))


class BlockEmu:
    def __init__(self, vi):
        T, D, NF, NCV, mode = ALL[vi]
        ring = vi >= len(gen_core.VARIANTS)
        tag, V0, FO, hs, _ = gen_core.gen_variant(T, D, NF, NCV, mode, ring)
        self.T, self.mode = T, mode
        text = gen_core.asm_text(T, D, NF, V0, FO, tag, hs, mode, ring)
        lines = [x.strip() for x in re.split(r'\\n\\t"?\s*"?', text)]
        self.ins, self.label, at, skip = [], {}, TEXT, False
        for x in lines:
            if x.startswith(".if"):
                skip = True
            elif x.startswith(".endif"):
                skip = False
            elif skip or not x:
                continue
            elif x.startswith(".p2align"):
                at = (at + 63) & ~63
            elif x.endswith(":"):
                self.label[x[:-1]] = at
            else:
                self.ins.append((at, x))
                at += gen_core.insn_bytes(x)
        self.at = {a: i for i, (a, _) in enumerate(self.ins)}
        self.end = at
        self.table = self.label[".Lgpx_table_%s" % tag]
        self.regions = []
        self.lds = np.zeros(64 * 1024, np.uint8)
        self.steps = 0

    # ---------------------------------------------------------------- memory
    def region(self, base, array):
        self.regions.append((base, base + array.nbytes, array.reshape(-1).view(np.uint8)))

    def bytes_at(self, addr, n):
        for lo, hi, b in self.regions:
            if lo <= addr and addr + n <= hi:
                return b[addr - lo: addr - lo + n]
        raise AssertionError("access of %d bytes at %#x is outside every buffer" % (n, addr))

    # ---------------------------------------------------------------- registers
    def sget(self, t, wide=False):
        t = t.strip()
        if t == "vcc":
            return self.vcc
        if t == "exec":
            return self.exec
        m = re.match(r"s\[(\d+):(\d+)\]$", t)
        if m:
            a = int(m.group(1))
            return self.s[a] | (self.s[a + 1] << 32)
        if re.match(r"s\d+$", t):
            return self.s[int(t[1:])]
        if "-.Lgpx" in t:
            a, b = t.split("-")
            return (self.label[a] - self.label[b]) & M32
        return int(t, 0) & (M64 if wide else M32)

    def sput(self, t, v):
        t = t.strip()
        m = re.match(r"s\[(\d+):(\d+)\]$", t)
        if t == "vcc":
            self.vcc = v & M64
        elif t == "exec":
            self.exec = v & M64
        elif m:
            a = int(m.group(1))
            self.s[a], self.s[a + 1] = v & M32, (v >> 32) & M32
        else:
            self.s[int(t[1:])] = v & M32

    def mask(self):
        return np.array([(self.exec >> k) & 1 for k in range(64)], bool)

    @staticmethod
    def bits(m):
        return int(sum(1 << int(k) for k in np.flatnonzero(m)))

    def vsrc(self, t, field, kind):
        """kind: u (uint32), f (float32), d (float64)"""
        t = t.strip()
        neg = ab = False
        if t.startswith("-") and ("v" in t or "s" in t):
            neg, t = True, t[1:]
        if t.startswith("|"):
            ab, t = True, t[1:-1]
        m = re.match(r"v\[?(\d+)", t)
        if m:
            r = int(m.group(1)) + (self.m0 if self.idx and field in self.modes else 0)
            if kind == "d":
                x = (self.v[r].astype(np.uint64) | (self.v[r + 1].astype(np.uint64) << np.uint64(32))).view(np.float64)
            else:
                x = self.v[r].copy()
        elif t == "vcc" or t.startswith("s"):
            val = self.sget(t)
            x = np.full(64, val, np.uint64).view(np.float64) if kind == "d" else np.full(64, val & M32, np.uint32)
        elif "." in t:
            x = np.full(64, float(t)) if kind == "d" else np.full(64, np.float32(float(t))).view(np.uint32)
        else:
            i = int(t, 0)
            if kind == "d":
                assert i == 0
                x = np.zeros(64)
            elif kind == "f" and not t.startswith("0x") and i != 0:
                raise AssertionError("integer inline constant in a float operand: " + t)
            else:
                x = np.full(64, i & M32, np.uint32)
        if kind == "f":
            x = x.view(np.float32)
        if ab:
            x = np.abs(x)
        return -x if neg else x

    def vput(self, t, x, pair=False):
        r = int(re.match(r"\s*v\[?(\d+)", t).group(1))
        if self.idx and "DST" in self.modes:
            r += self.m0
        m = self.mask()
        if x.dtype == np.float64:
            b = x.view(np.uint64)
            self.v[r][m] = (b & np.uint64(M32)).astype(np.uint32)[m]
            self.v[r + 1][m] = (b >> np.uint64(32)).astype(np.uint32)[m]
        else:
            self.v[r][m] = x.view(np.uint32)[m] if x.dtype == np.float32 else x.astype(np.uint32)[m]

    # ---------------------------------------------------------------- run
    def run(self, sgpr):
        self.s = [0xDEAD0000 + k for k in range(104)]
        for k, val in sgpr.items():
            self.s[k] = val & M32
        self.v = np.full((256, 64), 0x7FC00001, np.uint32)
        self.vcc, self.exec, self.scc, self.m0, self.idx, self.modes = 0, M64, 0, 0, False, set()
        pc = 0
        while pc < len(self.ins):
            addr, x = self.ins[pc]
            self.steps += 1
            assert self.steps < 3_000_000, "the block does not end"
            nxt = self.step(addr, x)
            pc = pc + 1 if nxt is None else (len(self.ins) if nxt == self.end else self.at[nxt])

    def jump(self, label):
        return self.label[label.strip()]

    def step(self, addr, x):
        op, _, rest = x.partition(" ")
        a = [t.strip() for t in rest.split(",")]
        if op in ("s_nop", "s_waitcnt", "s_barrier"):
            return None
        if op.startswith("s_"):
            return self.salu(addr, op, a, rest)
        if op.startswith("ds_"):
            return self.ds(op, rest)
        if op.startswith("global_"):
            return self.vmem(op, rest)
        return self.valu(op, a, rest)

    def salu(self, addr, op, a, rest):
        g = self.sget
        if op == "s_set_gpr_idx_on":
            r, modes = re.match(r"(s\d+), gpr_idx\(([A-Z0-9,]*)\)", rest).groups()
            self.idx, self.m0, self.modes = True, g(r) & 255, set(modes.split(","))
        elif op == "s_set_gpr_idx_off":
            self.idx = False
        elif op == "s_getpc_b64":
            self.sput(a[0], addr + 4)
        elif op == "s_setpc_b64":
            return g(a[0])
        elif op == "s_branch":
            return self.jump(a[0])
        elif op.startswith("s_cbranch_"):
            c = {"scc0": not self.scc, "scc1": self.scc, "vccnz": self.vcc != 0, "execz": self.exec == 0}[op[10:]]
            return self.jump(a[0]) if c else None
        elif op.startswith("s_load_dword"):
            n = 4 * int(op[len("s_load_dwordx"):] or 1) if "x" in op[7:] else 4
            off = g(a[2])
            src = self.bytes_at(g(a[1]) + off, n).view(np.uint32)
            r = int(re.match(r"s\[?(\d+)", a[0]).group(1))
            assert r % min(4, max(1, n // 4)) == 0
            for k in range(n // 4):
                self.s[r + k] = int(src[k])
        elif op.startswith("s_cmp_"):
            _, _, rel, ty = op.split("_")
            p, q = g(a[0]), g(a[1])
            if ty == "i32":
                p, q = (v - (1 << 32) if v >> 31 else v for v in (p, q))
            self.scc = {"eq": p == q, "lg": p != q, "lt": p < q, "le": p <= q, "gt": p > q, "ge": p >= q}[rel]
        elif op == "s_bitcmp1_b32":
            self.scc = bool((g(a[0]) >> g(a[1])) & 1)
        elif op in ("s_cselect_b32", "s_cselect_b64"):
            self.sput(a[0], g(a[1], op.endswith("64")) if self.scc else g(a[2], op.endswith("64")))
        elif op in ("s_mov_b32", "s_mov_b64"):
            self.sput(a[0], g(a[1], op.endswith("64")))
        else:
            p = g(a[1], "b64" in op)
            q = g(a[2], "b64" in op) if len(a) > 2 else 0
            sg = lambda v: v - (1 << 32) if v >> 31 else v   # noqa: E731
            if op == "s_add_u32":
                r = p + q
                self.scc = r >> 32 != 0
            elif op == "s_addc_u32":
                r = p + q + int(self.scc)
                self.scc = r >> 32 != 0
            elif op in ("s_sub_u32", "s_sub_i32"):
                r = p - q
                self.scc = r < 0 if op == "s_sub_u32" else self.scc
            elif op == "s_subb_u32":
                r = p - q - int(self.scc)
            elif op == "s_lshl_b32":
                r = p << (q & 31)
            elif op == "s_lshr_b32":
                r = p >> (q & 31)
            elif op in ("s_and_b32", "s_and_b64"):
                r = p & q
            elif op == "s_or_b64":
                r = p | q
            elif op == "s_xnor_b64":
                r = ~(p ^ q)
            elif op == "s_min_u32":
                r = min(p, q)
            elif op == "s_max_i32":
                r = max(sg(p), sg(q))
            elif op == "s_mul_i32":
                r = p * q
            elif op == "s_mul_hi_u32":
                r = (p * q) >> 32
            elif op == "s_bfe_u32":
                r = (p >> (q & 31)) & ((1 << ((q >> 16) & 127)) - 1)
            elif op == "s_bfm_b64":
                r = ((1 << (p & 63)) - 1) << (q & 63)
            elif op == "s_bcnt1_i32_b64":
                r = bin(g(a[1])).count("1")
            else:
                raise AssertionError(op)
            self.sput(a[0], r)
        return None

    def ds(self, op, rest):
        off = int(re.search(r"offset:(\d+)", rest).group(1)) if "offset" in rest else 0
        r = [int(t) for t in re.findall(r"v\[?(\d+)", rest.split(" offset")[0])]
        n = {"b64": 2, "b128": 4}[op.split("_")[2]]
        data, ad = (r[0], r[1]) if "read" in op else (r[1], r[0])
        m = self.mask()
        for lane in np.flatnonzero(m):
            p = int(self.v[ad][lane]) + off
            assert p % (4 * n) == 0 and p + 4 * n <= self.lds_used, (op, p)
            w = self.lds[p: p + 4 * n].view(np.uint32)
            for k in range(n):
                if "read" in op:
                    self.v[data + k][lane] = w[k]
                else:
                    w[k] = self.v[data + k][lane]

    def vmem(self, op, rest):
        off = int(re.search(r"offset:(\d+)", rest).group(1)) if "offset" in rest else 0
        assert off < 4096
        r = [int(t) for t in re.findall(r"v\[?(\d+)", rest.split(" offset")[0].replace("v[", "v"))]
        base = self.sget(re.search(r"s\[\d+:\d+\]", rest).group(0))
        n = 2 if "x2" in op else 1
        data, ad = (r[0], r[1]) if "load" in op else (r[1], r[0])
        for lane in np.flatnonzero(self.mask()):
            b = self.bytes_at(base + off + int(self.v[ad][lane]), 4 * n).view(np.uint32)
            for k in range(n):
                if "load" in op:
                    self.v[data + k][lane] = b[k]
                else:
                    b[k] = self.v[data + k][lane]

    def valu(self, op, a, rest):
        V, name = self.vsrc, re.sub(r"_e(32|64)$", "", op)
        with np.errstate(all="ignore"):
            if name.startswith("v_permlane"):
                w = 32 if "32" in name[:12] else 16
                p, q = (int(t[1:]) for t in a)
                assert self.exec == M64
                x, y = self.v[p].copy(), self.v[q].copy()
                for k in range(64):
                    if (k // w) % 2:
                        x[k], y[k - w] = self.v[q][k - w], self.v[p][k]
                self.v[p], self.v[q] = x, y
                return None
            if "dpp" in name:
                tail = rest.split("row_mask")[0]
                regs = [int(t) for t in re.findall(r"v(\d+)", tail)]
                ror = re.search(r"row_ror:(\d+)", tail)
                if ror:
                    src = (LANES & ~15) | ((LANES - int(ror.group(1))) & 15)
                else:
                    q = [int(t) for t in re.search(r"quad_perm:\[([\d,]+)\]", rest).group(1).split(",")]
                    src = (LANES & ~3) | np.array(q)[LANES & 3]
                assert self.exec == M64
                x = self.v[regs[1]][src]
                self.v[regs[0]] = x if "mov" in name else x + self.v[regs[2]]
                return None
            if name == "v_readlane_b32":
                self.sput(a[0], int(self.v[int(a[1][1:])][int(a[2])]))
                return None
            if name.startswith("v_cmp_"):
                _, _, rel, ty = name.split("_")
                kind = {"f32": "f", "u32": "u", "i32": "u"}[ty]
                p, q = V(a[1], "SRC0", kind), V(a[2], "SRC1", kind)
                r = {"lt": p < q, "gt": p > q, "eq": p == q, "neq": ~(p == q), "nlt": ~(p < q),
                     "u": np.isnan(p) | np.isnan(q) if kind == "f" else None}[rel]
                self.sput(a[0], self.bits(r & self.mask()))
                return None
            if name == "v_cndmask_b32":
                m = self.sget(a[3])
                m = np.array([(m >> k) & 1 for k in range(64)], bool)
                self.vput(a[0], np.where(m, V(a[2], "SRC1", "u"), V(a[1], "SRC0", "u")) if "." not in a[2] else
                          np.where(m, V(a[2], "SRC1", "f").view(np.uint32), V(a[1], "SRC0", "u")))
                return None
            if name.endswith("_f64") and not name.startswith("v_cvt") or name == "v_ldexp_f64":
                p = V(a[1], "SRC0", "d")
                if name == "v_ldexp_f64":
                    e = V(a[2], "SRC1", "u").view(np.int32) if a[2].startswith("v") else np.full(64, int(a[2]))
                    r = np.ldexp(p, e)
                elif name in ("v_floor_f64", "v_rndne_f64"):
                    r = np.floor(p) if "floor" in name else np.rint(p)
                else:
                    q = V(a[2], "SRC1", "d")
                    if name == "v_fma_f64":
                        c = V(a[3], "SRC2", "d")
                        r = fma(p, q, c)
                    else:
                        r = {"v_add_f64": p + q, "v_mul_f64": p * q, "v_max_f64": np.fmax(p, q)}[name]
                self.vput(a[0], r)
                return None
            if name.startswith("v_cvt_"):
                _, _, to, fr = name.split("_")
                if fr == "f64":
                    p = V(a[1], "SRC0", "d")
                    if to == "i32":
                        p = np.where(np.isnan(p), 0, np.clip(np.trunc(p), -2**31, 2**31 - 1)).astype(np.int64)
                        self.vput(a[0], (p & M32).astype(np.uint32))
                    else:
                        self.vput(a[0], p.astype(np.float32))
                elif fr == "f32":
                    self.vput(a[0], V(a[1], "SRC0", "f").astype(np.float64))
                else:
                    p = V(a[1], "SRC0", "u")
                    self.vput(a[0], (p.view(np.int32) if fr == "i32" else p).astype(np.float64))
                return None
            f = {"v_add_f32": lambda p, q: p + q, "v_sub_f32": lambda p, q: p - q, "v_subrev_f32": lambda p, q: q - p,
                 "v_mul_f32": lambda p, q: p * q, "v_max_f32": np.fmax, "v_min_f32": np.fmin,
                 "v_rndne_f32": None}
            if name in f:
                p = V(a[1], "SRC0", "f")
                self.vput(a[0], np.rint(p) if f[name] is None else f[name](p, V(a[2], "SRC1", "f")).astype(np.float32))
                return None
            if name in ("v_div_scale_f32", "v_rcp_f32", "v_fma_f32", "v_fmac_f32", "v_div_fmas_f32", "v_div_fixup_f32"):
                return self.division(name, a)
            p = V(a[1], "SRC0", "u").astype(np.uint64)
            q = V(a[2], "SRC1", "u").astype(np.uint64) if len(a) > 2 else None
            m32 = np.uint64(M32)
            if name == "v_mov_b32": r = p
            elif name == "v_add_u32": r = p + q
            elif name == "v_sub_u32": r = p - q
            elif name == "v_subrev_u32": r = q - p
            elif name == "v_max_u32": r = np.maximum(p, q)
            elif name == "v_mul_u32_u24": r = p * q
            elif name == "v_lshlrev_b32": r = q << (p & np.uint64(31))
            elif name == "v_lshrrev_b32": r = q >> (p & np.uint64(31))
            elif name == "v_ashrrev_i32": r = (q.astype(np.uint32).view(np.int32) >> (p & np.uint64(31)).astype(np.int32)).view(np.uint32).astype(np.uint64)
            elif name == "v_and_b32": r = p & q
            elif name == "v_or_b32": r = p | q
            elif name == "v_xor_b32": r = p ^ q
            elif name == "v_xnor_b32": r = ~(p ^ q)
            elif name == "v_lshl_add_u32": r = (p << q) + V(a[3], "SRC2", "u").astype(np.uint64)
            elif name == "v_bcnt_u32_b32": r = np.array([bin(int(t)).count("1") for t in p], np.uint64) + q
            elif name == "v_med3_i32":
                t = V(a[1], "SRC0", "u").view(np.int32)
                r = np.clip(t, int(a[2]), int(a[3])).astype(np.uint64)
            elif name in ("v_mbcnt_lo_u32_b32", "v_mbcnt_hi_u32_b32"):
                r = (np.minimum(LANES, 32) if "lo" in name else np.maximum(LANES - 32, 0)).astype(np.uint64) + q
            elif name == "v_bitop3_b32":
                tbl = int(re.search(r"bitop3:(\S+)", rest).group(1), 0)
                r = np.zeros(64, np.uint64)
                for i in range(8):
                    if (tbl >> i) & 1:
                        r |= (p if i & 4 else ~p) & (q if i & 2 else ~q) & (q if i & 1 else ~q)
            else:
                raise AssertionError(op)
            self.vput(a[0], (r & m32).astype(np.uint32))
        return None

    def division(self, name, a):
        """As in test_core_emulation: scaling is not modelled, the fix-up gives the IEEE quotient where it would act."""
        V, f64 = self.vsrc, np.float64
        if name == "v_div_scale_f32":
            self.vput(a[0], V(a[2], "SRC0", "f"))
            self.vcc = 0
        elif name == "v_rcp_f32":
            self.vput(a[0], (1.0 / V(a[1], "SRC0", "f").astype(f64)).astype(np.float32))
        elif name == "v_fmac_f32":
            p, q, c = V(a[1], "SRC0", "f"), V(a[2], "SRC1", "f"), V(a[0], "", "f")
            self.vput(a[0], (p.astype(f64) * q.astype(f64) + c.astype(f64)).astype(np.float32))
        elif name == "v_div_fixup_f32":
            q, den, num = V(a[1], "SRC0", "f"), V(a[2], "SRC1", "f"), V(a[3], "SRC2", "f")
            ieee = (num.astype(f64) / den.astype(f64)).astype(np.float32)
            big = lambda t: ~np.isfinite(t) | (t == 0) | (np.abs(t) > 2.0 ** 60) | (np.abs(t) < 2.0 ** -60)  # noqa: E731
            self.vput(a[0], np.where(big(num) | big(den) | big(q), ieee, q))
        else:
            p, q, c = (V(a[k], "SRC%d" % (k - 1), "f") for k in (1, 2, 3))
            self.vput(a[0], (p.astype(f64) * q.astype(f64) + c.astype(f64)).astype(np.float32))
        return None


KIND = {"sum_abs": 0, "mse": 1, "hits": 2, "cases": 3, "class_err": 4}


def emulate(vi, pop, X, y, kind, n_bits=0):
    """The block over every tile of X: partial sums (P, blocks), or outputs (P, N)."""
    emu = BlockEmu(vi)
    F, N = X.shape
    words, prog_off = gp.core_lower(pop, F, vi, emu.table)
    words = words.copy()
    P = pop.n_prog
    # rows and following lengths, as the library writes them for a group of consecutive programs
    ends = [int(prog_off[p + 1]) // 4 for p in range(P - 1)] + [(len(words) - 32) // 4]
    for p in range(P):
        nxt = ends[p + 1] - ends[p] if p + 1 < P else 0
        assert words[4 * (ends[p] - 1) + 2] & 0xFF000000 == 15 << 24
        words[4 * (ends[p] - 1) + 2] |= nxt
        words[4 * (ends[p] - 1) + 3] = p
    blocks = (N + 255) // 256
    part = np.full((P, blocks), np.nan)
    out = np.full((P, N), np.nan, np.float32)
    tab, coef = tables()
    emu.lds[:8 * len(tab)] = tab.view(np.uint8)
    lds_y = (8 * len(tab) + 15) // 16 * 16
    emu.lds_used = lds_y + 256 * emu.T
    for base, arr in ((CODE, words), (XBASE, X), (YBASE, y), (PART, part), (CASES, out), (COEF, coef)):
        emu.region(base, arr)
    W = 64 * emu.T
    for tile in range((N + W - 1) // W):
        left = min(W, N - tile * W)
        s = {63: 0, 62: 0, 78: 14, 86: F, 87: left, 92: blocks * 8, 93: KIND[kind], 96: ends[-1] * 16, 97: lds_y,
             98: min(32 * W, max(0, n_bits - 32 * tile * W)) if emu.mode == 2 else M32}
        for r, val in ((60, CODE), (82, XBASE + 4 * tile * W), (84, 4 * N), (88, YBASE + 4 * tile * W),
                       (90, PART + 8 * tile * (emu.T // 4)), (94, CASES + 4 * tile * W), (100, COEF)):
            s[r], s[r + 1] = val & M32, val >> 32
        emu.run(s)
    return out if kind == "cases" else part


def expected(o, y, kind, n_bits=0):
    """Partial sums by their definition, from the outputs o (P, N)."""
    P, N = o.shape
    blocks = (N + 255) // 256
    pad = blocks * 256 - N
    ok = np.pad(np.ones(N, bool), (0, pad))
    with np.errstate(all="ignore"):
        if n_bits:
            w = ~(o.view(np.uint32) ^ y.view(np.uint32)[None])
            left = np.clip(n_bits - 32 * np.arange(N), 0, 32)
            w &= np.array([(1 << int(k)) - 1 for k in left], np.uint32)
            t = np.array([[bin(int(v)).count("1") for v in r] for r in w], np.float64)
        elif kind == "hits":
            t = ((o > 0) == (y > 0)[None]).astype(np.float64)
        elif kind == "class_err":
            t = (~(np.rint(o) == y[None])).astype(np.float64)
        else:
            d = o - y[None]
            t = (d * d if kind == "mse" else np.abs(d)).astype(np.float64)
    t = np.where(ok[None], np.pad(t, ((0, 0), (0, pad))), 0.0).reshape(P, blocks, 4, 64)
    v = np.zeros((P, blocks, 64))
    for j in range(4):
        v = v + t[:, :, j]
    for step in (32, 16, 8, 4, 2, 1):
        v = v + v[:, :, LANES ^ step]
    return v[:, :, 0]


def same(a, b):
    return ((a == b) | (np.isnan(a) & np.isnan(b))).all()


REAL = [i for i, v in enumerate(ALL) if v[4] != 2]
BOOL = [i for i, v in enumerate(ALL) if v[4] == 2]
SETS = {0: synth.FULL, 1: synth.BASIC, 3: synth.SHUTTLE_SET, 4: synth.KDD_SET}


@pytest.mark.parametrize("vi", REAL)
def test_block_programs_and_fitness(vi):
    """A unit of several programs, full and ragged tiles, with each fitness kind on a different size."""
    T, D, NF, NCV, mode = ALL[vi]
    F = min(NF, 9 if vi % 2 else 3)
    rng = synth.rng_for(700 + vi)
    pop = synth.ptc2_population(rng, 6, SETS[mode], F, 1, 60, 0.2)
    for kind, N in (("mse", 64 * T + 37), ("sum_abs", 64 * T - 1), ("hits", 64 * T + 256), ("class_err", 1),
                    ("cases", 64 * T + 65)):
        X = synth.uniform_cases(rng, F, N, -3, 3)
        y = np.round(synth.uniform_cases(rng, 1, N, -2, 2)[0])
        o = oracle.tree_outputs(pop.tok, pop.cst, pop.off, X)
        got = emulate(vi, pop, X, y, kind)
        assert same(got, o) if kind == "cases" else same(got, expected(o, y, kind)), kind


@pytest.mark.parametrize("vi", BOOL)
def test_block_boolean_hits(vi):
    T, D, NF, NCV, _ = ALL[vi]
    F = min(NF, 7)
    rng = synth.rng_for(800 + vi)
    pop = synth.ptc2_population(rng, 5, synth.BOOL_SET, F, 1, 60, 0.0)
    for N, n_bits in ((64 * T + 3, (64 * T + 2) * 32 + 5), (64 * T, 64 * T * 32), (1, 1)):
        X = rng.integers(0, 2**32, size=(F, N), dtype=np.uint64).astype(np.uint32)
        y = rng.integers(0, 2**32, size=N, dtype=np.uint64).astype(np.uint32)
        o = oracle.bool_outputs(pop.tok, pop.off, X).view(np.float32)
        got = emulate(vi, pop, X.view(np.float32), y.view(np.float32), "hits", n_bits)
        assert same(got, expected(o, y.view(np.float32), "hits", n_bits))


@pytest.mark.parametrize("vi", [i for i in REAL if ALL[i][4] in (0, 4)])
def test_block_transcendentals(vi):
    """sin, cos, exp and log of ordinary, large, tiny and special arguments, of a variable and in place on the stack.
    The emulated fused operation may round a tie twice, so one ulp is allowed now and then."""
    T = ALL[vi][0]
    from tests import progs
    exprs = ["(%s x0)" % f for f in ("sin", "cos", "exp", "log")] + \
            ["(%s (* x0 x1))" % f for f in ("sin", "cos", "exp", "log")] + ["(sin 0.75)", "(log (exp (cos x0)))"]
    pop = progs.pop(*exprs)
    rng = synth.rng_for(900 + vi)
    N = 2 * 64 * T
    X = synth.uniform_cases(rng, 2, N, -20, 20)
    X[0, :96] = rng.integers(0, 2**32, 96, dtype=np.uint64).astype(np.uint32).view(np.float32)
    X[0, 96:116] = [0.0, -0.0, 1e-45, -1e-45, 1e-6, 9.99999997e-7, np.inf, -np.inf, np.nan, 88.0, 88.5, -104.0, -103.95,
                    1.7592186e13, 1.7592185e13, -2.0e13, 3.4e38, -3.4e38, 1e20, 2.4414e-4]
    X[1, :N // 2] = 1.0
    y = np.zeros(N, np.float32)
    o = oracle.tree_outputs(pop.tok, pop.cst, pop.off, X)
    got = emulate(vi, pop, X, y, "cases")
    gi, oi = got.view(np.int32).astype(np.int64), o.view(np.int32).astype(np.int64)
    exact = (gi == oi) | (np.isnan(got) & np.isnan(o))
    assert (exact | (np.abs(gi - oi) <= 1)).all(), np.argwhere(~exact)[:5]
    assert exact.mean() > 0.999


@pytest.mark.parametrize("vi", [i for i in REAL if i >= len(gen_core.VARIANTS)])
def test_ring_core_operand_forms(vi):
    """Every operand form of division, the compares, AND, OR and IF on a ring core, at the lowest and at the highest
    levels the core has (where a variable has no level above it to be copied to), with protected divisors, signed
    zeros, NaN and equal operands among the cases: the oracle's bits."""
    T, D, NF, NCV, mode = ALL[vi]
    F = min(NF, 3)
    x = lambda k: "x%d" % (k % F)   # noqa: E731
    ops = ("/", ">", "<", "==", "and", "or")

    def deep(e, levels):
        """e evaluated with `levels` values below it on the stack: each partner is a tree that needs as many levels."""
        full = lambda n: x(n) if n == 0 else "(+ %s %s)" % (full(n - 1), full(n - 1))   # noqa: E731
        for n in range(levels):
            e = "(- %s %s)" % (full(D - 1 - (levels - 1 - n)), e)
        return e
    exprs = []
    for f in ops:
        p, q = "(+ %s %s)" % (x(0), x(2)), "(* %s %s)" % (x(1), x(2))
        exprs += ["(%s %s %s)" % (f, a, b) for a, b in (
            (p, q), (p, "(+ %s (* %s %s))" % (x(0), q, p)), ("(- %s (* %s %s))" % (x(1), q, p), p), (p, x(1)), (x(1), q),
            (x(0), x(1)), (x(1), x(1)), (p, "0.5"), ("-0.0", q), (x(0), "2"), ("0.25", x(1)))]
        exprs += [deep("(%s (+ %s 0.5) %s)" % (f, x(0), x(1)), n) for n in (1, 2)]
    exprs += ["(if %s %s %s)" % (x(0), x(1), x(2)), "(if (> %s %s) (* %s 3) -1.5)" % (x(0), x(1), x(2)),
              "(if (+ %s 1) (* (- %s %s) (+ %s %s)) %s)" % (x(0), x(1), x(2), x(1), x(0), x(1)),
              "(if %s (* (- %s %s) (+ %s %s)) (- 1 %s))" % (x(0), x(1), x(2), x(1), x(0), x(1)),
              "(if (- 1 %s) %s (* (- %s %s) (+ %s %s)))" % (x(0), x(1), x(1), x(2), x(1), x(0))]
    from tests import progs
    pop = progs.pop(*exprs)
    N = 64 * T + 19
    X = np.round(synth.uniform_cases(synth.rng_for(950 + vi), F, N, -2, 2))
    X[0, ::7] = -0.0
    X[F - 1, 1::9] = np.nan
    X[0, 2::11] = 5e-7
    o = oracle.tree_outputs(pop.tok, pop.cst, pop.off, X)
    got = emulate(vi, pop, X, np.zeros(N, np.float32), "cases")
    bad = np.argwhere(~((got.view(np.int32) == o.view(np.int32)) | (np.isnan(got) & np.isnan(o))))
    assert not len(bad), (exprs[bad[0][0]], got[tuple(bad[0])], o[tuple(bad[0])])


@pytest.mark.parametrize("vi", [i for i in REAL if ALL[i][4] == 4 and i >= len(gen_core.VARIANTS)])
def test_rows_are_computed_and_pushed(vi):
    """A unit with rows: the programs that compute them (sin, exp and cos of features, to LDS) run first, then the
    wave's own, which push them at two levels in every phase and go on; a wave without programs ends after its rows.
    LDS beyond the rows stays as it was."""
    T, D, NF, NCV, mode = ALL[vi]
    emu = BlockEmu(vi)
    tag, V0, FO, hs, _ = gen_core.gen_variant(T, D, NF, NCV, mode, True)
    K, ph = gen_core.K, gen_core.RING_PHASE
    slot = {(h.kind, h.op, h.p1, h.p2): emu.table + h.slot * gen_core.RING_SLOT for h in hs}
    base = gen_core.rows_base(T, D, NF, NCV, mode)

    def records(*items):
        """(kind, op, p1, payload, constant), phases in turn from 0, again from 0 after a function's exit"""
        out, k = [], 0
        for kind, op, p1, pay, cst in items:
            a = slot[(K[kind] | (k << ph), op, p1, 0)]
            out.append((a & M32, a >> 32, pay, cst))
            k = 0 if kind == "EXIT" else (k + 1) & 3
        return out
    F, N = 3, 64 * T - 5
    fx = lambda f: FO + f * T   # noqa: E731
    rows = [(4, 0), (6, 2), (5, 1)]
    own = [records(("PUSHR", 0, 0, 256 * T * 1, 0), ("PUSHR", 0, 1, 256 * T * 2, 0), ("SS", 0, 0, 0, 0), ("PUSHR", 0, 1, 0, 0),
                   ("SS", 2, 0, 0, 0), ("PUSHR", 0, 1, 256 * T * 1, 0), ("SS", 1, 0, 0, 0), ("EXIT", 0, 0, 15 << 24 | 2, 0)),
           records(("PUSHR", 0, 0, 0, 0), ("EXIT", 0, 0, 15 << 24, 1))]
    derived = [records(("EXIT", 0, 0, fx(f) | op << 24, 0), ("EXIT", 0, 0, 15 << 24 | 2, r)) for r, (op, f) in enumerate(rows)]
    code = sum(own, []) + sum(derived, [])
    words = np.array(code + [(0, 0, 0, 0)] * 8, np.uint64).astype(np.uint32).reshape(-1)
    n_own = sum(len(p) for p in own)
    X = synth.uniform_cases(synth.rng_for(40 + vi), F, N, -2, 2)
    y = np.zeros(N, np.float32)
    out = np.full((2, N), np.nan, np.float32)
    tab, coef = tables()
    emu.lds[:] = 0xA5
    emu.lds[:8 * len(tab)] = tab.view(np.uint8)
    emu.lds_used = base + 256 * T * len(rows)
    for b, arr in ((CODE, words), (XBASE, X), (YBASE, y), (CASES, out), (COEF, coef), (PART, np.zeros((2, 1)))):
        emu.region(b, arr)
    s = {63: 0, 62: 16 * n_own, 78: 14, 86: F, 87: N, 92: 8, 93: gen_core.TO_ROW, 96: 16 * len(code), 97: 8 * len(tab),
         56: 0, 57: 16 * n_own, 98: KIND["cases"]}
    for r, val in ((60, CODE), (82, XBASE), (84, 4 * N), (88, YBASE), (90, PART), (94, CASES), (100, COEF)):
        s[r], s[r + 1] = val & M32, val >> 32
    emu.run(dict(s))
    f = [np.array([oracle.apply(op, v) for v in X[k]], np.float32) for op, k in rows]
    want = np.stack([(f[1] + f[2]) * f[0] - f[1], f[0]]).astype(np.float32)
    assert np.abs(out.view(np.int32).astype(np.int64) - want.view(np.int32)).max() <= 1
    assert (emu.lds[emu.lds_used:] == 0xA5).all()
    out[:] = np.nan
    emu.run(dict(s, **{}) | {56: 16 * n_own, 57: 16 * n_own})     # no programs of its own
    assert np.isnan(out).all()


@pytest.mark.parametrize("vi", [i for i in REAL if ALL[i] in gen_core.WIDE])
@pytest.mark.parametrize("N", [1, 64, 200, 256])
def test_features_in_lds(vi, N):
    """A unit whose features lie in LDS beyond those in registers: the programs of the rows load them (nothing is read
    past the data), as they are and as operands of functions, and the wave's own programs push them."""
    T, D, NF, NCV, mode = ALL[vi]
    emu = BlockEmu(vi)
    tag, V0, FO, hs, _ = gen_core.gen_variant(T, D, NF, NCV, mode, True)
    K, ph = gen_core.K, gen_core.RING_PHASE
    slot = {(h.kind, h.op, h.p1, h.p2): emu.table + h.slot * gen_core.RING_SLOT for h in hs}
    base = gen_core.rows_base(T, D, NF, NCV, mode)

    def records(*items):
        out, k = [], 0
        for kind, op, p1, pay, cst in items:
            a = slot[(K[kind] | (k << ph), op, p1, 0)]
            out.append((a & M32, a >> 32, pay, cst))
            k = 0 if kind == "EXIT" else (k + 1) & 3
        return out
    F = NF + 3
    load = lambda f: ("EXIT", 0, 0, 14 << 24 | f, 0)   # noqa: E731
    end = lambda r, n: ("EXIT", 0, 0, 15 << 24 | n, r)   # noqa: E731
    own = [records(("PUSHR", 0, 0, 0, 0), ("PUSHR", 0, 1, 256 * T, 0), ("SS", 1, 0, 0, 0), ("PUSHR", 0, 1, 512 * T, 0),
                   ("SS", 2, 0, 0, 0), ("SX", 0, 0, FO, 0), end(0, 0))]
    derived = [records(load(F - 1), end(0, 2)), records(load(NF), end(1, 3)),
               records(load(F - 2), ("EXIT", 0, 0, 4 << 24, 0), end(2, 0))]
    code = sum(own, []) + sum(derived, [])
    words = np.array(code + [(0, 0, 0, 0)] * 8, np.uint64).astype(np.uint32).reshape(-1)
    X = synth.uniform_cases(synth.rng_for(70 + vi), F, N, -2, 2)
    out = np.full((1, N), np.nan, np.float32)
    tab, coef = tables()
    emu.lds[:] = 0xA5
    emu.lds[:8 * len(tab)] = tab.view(np.uint8)
    emu.lds_used = base + 256 * T * 3
    for b, arr in ((CODE, words), (XBASE, X), (YBASE, np.zeros(N, np.float32)), (CASES, out), (COEF, coef),
                   (PART, np.zeros((1, 1)))):
        emu.region(b, arr)
    s = {63: 0, 62: 16 * len(own[0]), 78: 14, 86: NF, 87: N, 92: 8, 93: gen_core.TO_ROW, 96: 16 * len(code), 97: 8 * len(tab),
         56: 0, 57: 16 * len(own[0]), 98: KIND["cases"]}
    for r, val in ((60, CODE), (82, XBASE), (84, 4 * N), (88, YBASE), (90, PART), (94, CASES), (100, COEF)):
        s[r], s[r + 1] = val & M32, val >> 32
    emu.run(s)
    sin = np.array([oracle.apply(4, v) for v in X[F - 2]], np.float32)
    prod = ((X[F - 1] - X[NF]) * sin).astype(np.float32)
    want = (prod + X[0]).astype(np.float32)
    # the sine may be off by a unit of its last place, the product by two then, and the sum is rounded once more
    assert (np.abs(out[0] - want) <= 2 * np.spacing(np.abs(prod)) + np.spacing(np.abs(want))).all()
    assert (emu.lds[emu.lds_used:] == 0xA5).all()
