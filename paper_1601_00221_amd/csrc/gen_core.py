"""Generate the hand-written gfx950 interpreter core (a build step).

    python gen_core.py OUT_DIR

Writes ``core_gen.inc`` (the tables that name every variant's handlers), one
``core_v_*.hip`` a kernel variant (T case slots per lane, D stack levels, NF
feature slots) with its inline-asm block, and ``core_dispatch.inc``.

Design.  The whole two-dimensional stack (level l, slot j), the registers of
a linear program and the wave's case tile live in a VGPR range the compiler
does not allocate (the kernel caps the compiler's own VGPRs).  Offsets in
that range, relative to its first register V0:

    stack level l / linear register r, slot j :  l*T + j        (l < RB)
    feature f, slot j                          :  RB*T + f*T + j  (f < NF)

with RB = max(8, D) register/stack levels (RB = D in the Boolean kernels,
which run trees only).

A program is a list of 16-byte instructions

    dword 0-1  absolute address of the handler that executes it
    dword 2    operand offsets (byte 0 = first index, byte 1 = second index;
               for an exit: A, B, destination offsets and the operation)
    dword 3    constant operand (binary32 bits)

A handler executes its own T vector instructions with the wave-uniform
operand offset applied through the gfx9 VGPR index mode (one index per
instruction; the other operands of the handler are fixed registers, so
handlers are specialised on stack level or register number) and jumps to the
next handler's address.  Every lane runs the same program, so the jump is
uniform.  Records are loaded ahead: two at a time by pair cores, whose
handlers come in two phases; in ring cores four lie in s[b:b+15], handlers
come in four phases, and each waits only for the pair that was requested two
instructions before.

The block runs a whole unit.  It loads the tile (features into VGPRs, targets
into LDS), computes the block's share of the tile's rows, and runs the unit's
programs one after another: protected division and the classification
functions in handlers of their own, sin/cos/exp/log in the block's tail
(transc), and at the end of a program, which is an exit with operation 15,
the fitness terms and their sum over the wave (program_end), while the next
program's first records and code lines are already under way.

SGPRs used by the block: s[60:61] code base, s62 byte offset of the record
loaded next, s63 probe flag, s[64:71] the records of pair cores, s[36:51] or
s[8:23] those of ring cores (ring_base), s[66:67] an exit's payload and
constant, s72-s77, s79-s81 temporaries (s[76:77] also the return of a shared
body and, when probed, the table's address), s78 code lines fetched at a time,
s[58:59] and s99 the lines still to fetch, s[82:85] X and its stride, s86
features, s87 cases left in the tile, s[88:95] y, partials, their stride and
the outputs, s93 the fitness kind, s96 the end of the unit's records, s97 the
targets in LDS, s98 bits left (Boolean) or the kind after the rows, s56 and
s57 the wave's own records meanwhile, s[24:55] and s[100:101] coefficients.
"""
import os
import sys

SLOT = 64                 # bytes per handler slot; longer handlers take several
LIN_REGS = 8              # register slots reserved for linear programs (and stack levels)

# (T, D, NF, NCV, MODE) variants: T case slots per lane, D stack levels, NF
# feature slots, NCV VGPRs left to the compiler (the core owns v[NCV ...]),
# MODE = 0 for the arithmetic function set with the sin/cos/exp/log code,
# 1 without that code (for programs that use none), 2 for the Boolean function set (slots are
# 32-bit words of bit-packed cases), 3 like 1 for trees only (no linear
# handlers or registers: a handler table half the size, and the stack
# levels start the VGPR range), 4 like 0 for trees only (the core of mode
# 3 with the sin/cos/exp/log code).  sin/cos/exp/log (binary64) run in the
# registers below the core's: from 48 on two slots side by side, from 64 on
# with the constants kept.
VARIANTS = [
    (8, 6, 8, 40, 0),
    (8, 6, 8, 128, 0),
    (8, 8, 8, 40, 0),
    (4, 8, 8, 40, 0),
    (4, 8, 16, 40, 0),
    (4, 12, 32, 40, 0),
    (8, 8, 8, 128, 0),
    (4, 8, 16, 128, 0),
    (4, 12, 32, 80, 0),
    (4, 8, 8, 64, 0),
    (4, 8, 8, 96, 0),
    (4, 8, 16, 64, 0),
    (8, 6, 8, 40, 1),
    (8, 8, 8, 40, 1),
    (4, 8, 16, 40, 1),
    (4, 12, 32, 40, 1),
    (8, 6, 8, 56, 3),
    (8, 8, 8, 40, 3),
    (4, 8, 16, 48, 3),
    (4, 8, 44, 48, 4),
    (8, 6, 20, 48, 2),
    (8, 8, 20, 32, 2),
    (4, 12, 32, 40, 2),
    # deep programs: every tree of at most GP_MAX_LEN nodes needs at most 20
    # levels (15 without IF), 16 for the binary Boolean set; with more than 32
    # features the deepest that fits beside them is 12
    (4, 20, 32, 40, 0),
    (4, 12, 44, 32, 4),
    (4, 16, 32, 40, 2),
    (4, 6, 20, 24, 2),
    (4, 8, 12, 48, 3),
    # 4 waves per SIMD at T = 4: register programs over 16 features (13 % faster than (4, 8, 16, 40))
    (4, 8, 16, 32, 1),
]

# A kernel's place in VARIANTS + RING_VARIANTS is its number in the interface (gp_batch_config, GP2D_VARIANT), which
# programs store: kernels are added at the end and keep their places.  These are kept for configurations that name
# them: ring cores (and (4, 9, 11, 48), below) took their place in the default choice.
BY_NUMBER_ONLY = {(8, 6, 8, 56, 3), (8, 8, 8, 40, 3), (4, 8, 16, 48, 3), (4, 8, 44, 48, 4), (8, 6, 20, 48, 2),
                  (8, 8, 20, 32, 2), (4, 6, 20, 24, 2), (4, 8, 12, 48, 3)}

# Variants on ring cores (below): trees of functions that stay in the core, whose instructions are short enough for
# the scalar cache's latency to show.  5 levels hold the benchmark populations of up to 256 nodes without IF; the
# compiled code needs few registers, so 128 of them (4 waves per SIMD) hold T = 8 over 8 features: 0.631 ms on the
# {+,-,*} workload against 0.711 with 3 waves, both before the ring.
RING_VARIANTS = [
    (8, 5, 8, 24, 3),
    (8, 8, 8, 24, 3),
    (8, 5, 4, 24, 3),
    (8, 6, 2, 24, 3),
    (4, 6, 12, 24, 3),
    (4, 8, 16, 24, 3),
    (4, 6, 24, 24, 3),
    (4, 8, 44, 24, 3),
    (8, 6, 12, 16, 2),
    (4, 6, 20, 16, 2),
    (4, 8, 20, 16, 2),
    (4, 8, 8, 64, 4),
    (4, 6, 12, 56, 4),
    (4, 8, 16, 56, 4),
    (4, 9, 11, 48, 4),
]

# Ring cores with sin/cos/exp/log that hold more features than their registers do: the others lie in LDS, as rows that
# a block loads for its tile and its programs push.  The value is how many features they take.  44 features in registers
# leave room for 2 waves a SIMD, which kept the vector units busy 66 % of the time; 11 leave room for 4, two blocks a CU:
# 46.8 -> 38.8 ms on 4096 classification trees over 41 features x 494021 cases, though a third of the functions' rows
# give way to features and every operand in LDS takes a record.  (One block of 16 waves a CU, with room for all the
# rows: 43.9 ms; its waves wait for the slowest of them, and nothing else runs meanwhile.)
WIDE = {(4, 9, 11, 48, 4): 44}


def vname(v):
    """Kernel name suffix of a variant: T_D_NF_NCV, plus _a when it has no
    sin/cos/exp/log code, _at when it also runs trees only, _t for trees only
    with that code, and _b for the Boolean function set."""
    return "%d_%d_%d_%d%s" % (v[0], v[1], v[2], v[3], ("", "_a", "_b", "_at", "_t")[v[4]])

OPS = {"add": "v_add_f32_e32", "sub": "v_sub_f32_e32", "mul": "v_mul_f32_e32"}
OP_ID = {"add": 0, "sub": 1, "mul": 2}
# Boolean functions (ids as the tree opcodes GP_AND .. GP_NOR).  AND and OR
# are one VOP2 operation; NAND and NOR one v_bitop3_b32, whose truth table
# has bit (4 s0 + 2 s1 + s2) set where the result is 1 (the third source is
# ignored by these tables).
BOOL_OPS = {"and": "v_and_b32_e32", "or": "v_or_b32_e32", "nand": 0x3F, "nor": 0x03}
BOOL_ID = {"and": 8, "or": 9, "nand": 10, "nor": 11}


def bool_op(op, d, a, b):
    """d = a op b; a and b keep their positions as first and second source."""
    ins = BOOL_OPS[op]
    if isinstance(ins, str):
        return "%s %s, %s, %s" % (ins, d, a, b)
    return "v_bitop3_b32 %s, %s, %s, %s bitop3:0x%x" % (d, a, b, b, ins)


def xx_levels(D, NF, mode, ring):
    """Levels at which two variables are pushed in one pass, by a handler for
    every distance between them: all of them over up to 8 features (a deep
    ring core keeps to the lowest three, so that its table stays within a
    branch's reach), the lowest two in Boolean ring cores, where most are."""
    if mode == 2:
        return 2 if ring else 0
    return 0 if NF > 8 else 3 if ring and D > 6 else D


def waves_per_block(T, D, NF, NCV, mode, ring):
    """Four; eight in ring cores with sin/cos/exp/log whose occupancy eight
    divides: the waves of a block share the rows of its tile in LDS, and a
    wider block has room for more of them.  Half of what a CU holds where features lie in LDS."""
    simd = 512 // ((NCV + (reg_levels(D, mode) + NF) * T + 7) // 8 * 8)
    if (T, D, NF, NCV, mode) in WIDE and ring:
        return 2 * simd
    return 8 if ring and mode == 4 and simd % 2 == 0 else 4


def rows_base(T, D, NF, NCV, mode):
    """LDS address of a block's rows: behind the reduction tables and each wave's targets."""
    return LDS_PI + 8 * 8 + 256 * T * waves_per_block(T, D, NF, NCV, mode, True)


def row_address(V0):
    """The register that holds a lane's offset in a row."""
    return V0 - work_regs(V0, 4, True)


def reg_levels(D, mode):
    """Register/stack levels before the features: linear programs need
    LIN_REGS registers; Boolean and trees-only kernels have none."""
    return D if mode >= 2 else max(LIN_REGS, D)

# handler kinds (keep in sync with the generated enum below)
KINDS = ["EXIT", "SS", "SSR", "SX", "XS", "SC", "CS", "XX", "XX2", "XC", "CX", "PUSHX", "PUSHC",
         "RR", "XR", "FF", "CR", "RC", "MOVC", "MOVX", "DVV", "DVC", "DCV", "CVV", "CVC", "CCV", "IF3",
         # ring cores: compares and logic of two stack entries or of one and a variable, divisions with a stack entry
         "CSS", "CSX", "DSS", "DSSR", "DSX", "DXS",
         # ring cores with sin/cos/exp/log: push a row that the block has computed for its tile
         "PUSHR"]
# Protected division runs in the core: a / b with a and b at any two offsets
# (DVV), b the constant (DVC) or a the constant (DCV), the result to a third
# offset.  Its temporaries are the last DIV_TMP registers of the compiler's
# range (clobbered by the block), its flags vcc, its indexes s73/s74/s79 and
# the protection threshold s80.
DIV_TMP = 7
DIV_THRESHOLD = 0x358637BD       # 1e-6f: |b| below it gives 1
K = {k: i for i, k in enumerate(KINDS)}


def vr(n):
    assert 0 <= n < 256, n
    return "v%d" % n


VOP3_ONLY = ("v_bitop3", "v_div_scale_f32", "v_fma_f32", "v_div_fmas_f32", "v_div_fixup_f32")


def insn_bytes(text):
    """Encoded size of an instruction the handlers use: scalar loads, VOP3
    encodings and a scalar move of a literal take 8 bytes, everything else 4."""
    if text.startswith(("s_load", "ds_") + VOP3_ONLY) or text.split(" ")[0].endswith("_e64"):
        return 8
    if text.startswith("s_mov_b32") and "0x" in text:
        return 8
    return 4


class Handler:
    def __init__(self, kind, op=0, p1=0, p2=0):
        self.kind, self.op, self.p1, self.p2 = kind, op, p1, p2
        self.lines = []
        self.size = 0
        self.phases = None      # (phase A lines, phase B lines) of a handler written per phase
        self.body = None        # its operation, a function of the registers that hold its offsets and constant
        self.n_idx = 0          # and the number of those offsets
        self.then = None        # ring cores: a shared body that the handler goes on to
        self.row = None         # a push of a row: its first register, the lane's offset, a temporary, the rows' LDS address

    def emit(self, text, nbytes):
        self.lines.append(text)
        self.size += nbytes


def gen_variant(T, D, NF, NCV, mode=0, ring=False):
    V0 = NCV
    FO = reg_levels(D, mode) * T       # register/stack block, then the features
    assert FO + NF * T <= 256, "index range exceeds 8 bits"
    assert V0 + FO + NF * T <= 256
    assert NCV % 8 == 0
    tag = "T%dD%dF%dV%d%s" % (T, D, NF, NCV, {2: "B", 3: "R", 4: "R"}.get(mode, ""))
    hs = []

    def prologue(h, const=False, second_index=False, index=None):
        """Save what the handler still needs from the current record (the
        next record's load overwrites s[64:67]), then start that load.  A
        handler with one index turns the index mode on straight from the
        payload, before the load is issued."""
        if const:
            h.emit("s_mov_b32 s72, s67", 4)
        if index == "off":
            h.emit("s_set_gpr_idx_off", 4)
        elif index is not None:
            idx_on(h, "s66", index)
        else:
            h.emit("s_mov_b32 s70, s66", 4)
        if second_index:
            h.emit("s_lshr_b32 s71, s66, 8", 4)
        h.emit("s_add_u32 s62, s62, 16", 4)
        h.emit("s_load_dwordx4 s[64:67], s[60:61], s62", 8)

    def idx_on(h, sreg, modes):
        h.emit("s_set_gpr_idx_on %s, gpr_idx(%s)" % (sreg, ",".join(modes)), 4)

    def epilogue(h):
        h.emit("s_waitcnt lgkmcnt(0)", 4)
        h.emit("s_setpc_b64 s[64:65]", 4)

    def valu(h, text):
        h.emit(text, insn_bytes(text))

    # ---------------------------------------------------------------- exit
    h = Handler(K["EXIT"])
    h.emit("s_set_gpr_idx_off", 4)
    h.emit("s_branch .Lgpx_end_%s" % tag, 4)
    hs.append(h)

    if mode == 2:
        bool_handlers(hs, T, D, V0, FO, prologue, idx_on, epilogue, valu)
        if ring:
            # two variables in one pass (as XX above), at the levels where most of them are pushed
            for op in BOOL_OPS:
                for l in range(xx_levels(D, NF, mode, ring)):
                    for dl in range(NF):
                        h = Handler(K["XX"], BOOL_ID[op], l, dl)
                        prologue(h, index=["SRC0", "SRC1"])
                        for j in range(T):
                            valu(h, bool_op(op, vr(V0 + l * T + j), vr(V0 + FO + j), vr(V0 + FO + dl * T + j)))
                        epilogue(h)
                        hs.append(h)
        return finish(hs, tag, V0, FO, ring, mode)

    # ---------------------------------------------------------------- trees
    for op in ("add", "sub", "mul"):
        h = Handler(K["SS"], OP_ID[op])            # s[h-2] = s[h-2] op s[h-1]; index (h-2)*T
        prologue(h, index=["SRC0", "SRC1", "DST"])
        for j in range(T):
            valu(h, "%s %s, %s, %s" % (OPS[op], vr(V0 + j), vr(V0 + j), vr(V0 + T + j)))
        epilogue(h)
        hs.append(h)
    h = Handler(K["SSR"], OP_ID["sub"])            # s[h-2] = s[h-1] - s[h-2]
    prologue(h, index=["SRC0", "SRC1", "DST"])
    for j in range(T):
        valu(h, "v_sub_f32_e32 %s, %s, %s" % (vr(V0 + j), vr(V0 + T + j), vr(V0 + j)))
    epilogue(h)
    hs.append(h)
    for op in ("add", "sub", "mul"):
        for l in range(D):
            h = Handler(K["SX"], OP_ID[op], l)     # s[l] = s[l] op x[b]; index = feature offset
            prologue(h, index=["SRC1"])
            for j in range(T):
                r = vr(V0 + l * T + j)
                valu(h, "%s %s, %s, %s" % (OPS[op], r, r, vr(V0 + j)))
            epilogue(h)
            hs.append(h)
    for l in range(D):
        h = Handler(K["XS"], OP_ID["sub"], l)      # s[l] = x[a] - s[l]
        prologue(h, index=["SRC0"])
        for j in range(T):
            r = vr(V0 + l * T + j)
            valu(h, "v_sub_f32_e32 %s, %s, %s" % (r, vr(V0 + j), r))
        epilogue(h)
        hs.append(h)
    for op, ins in (("add", "v_add_f32_e32"), ("mul", "v_mul_f32_e32"), ("sub", "v_subrev_f32_e32")):
        h = Handler(K["SC"], OP_ID[op])            # s[l] = s[l] op c; index l*T
        prologue(h, const=True, index=["SRC1", "DST"])
        for j in range(T):
            valu(h, "%s %s, s72, %s" % (ins, vr(V0 + j), vr(V0 + j)))
        epilogue(h)
        hs.append(h)
    h = Handler(K["CS"], OP_ID["sub"])             # s[l] = c - s[l]
    prologue(h, const=True, index=["SRC1", "DST"])
    for j in range(T):
        valu(h, "v_sub_f32_e32 %s, s72, %s" % (vr(V0 + j), vr(V0 + j)))
    epilogue(h)
    hs.append(h)
    if NF <= 8:
        # push x[a] op x[b] at level l: both sources relative to one index a*T,
        # the second one displaced by delta = b - a feature rows
        for op in ("add", "mul", "sub"):
            deltas = range(0, NF) if op != "sub" else range(-(NF - 1), NF)
            for l in range(xx_levels(D, NF, mode, ring)):
                for dl in deltas:
                    h = Handler(K["XX"], OP_ID[op], l, dl)
                    prologue(h, index=["SRC0", "SRC1"])
                    for j in range(T):
                        valu(h, "%s %s, %s, %s" % (OPS[op], vr(V0 + l * T + j), vr(V0 + FO + j),
                                                   vr(V0 + FO + dl * T + j)))
                    epilogue(h)
                    hs.append(h)
    for op in ("add", "sub", "mul"):
        for l in range(D):
            h = Handler(K["XX2"], OP_ID[op], l)    # two passes: s[l] = x[b]; s[l] = x[a] op s[l]
            prologue(h, second_index=True)
            idx_on(h, "s71", ["SRC0"])
            for j in range(T):
                valu(h, "v_mov_b32_e32 %s, %s" % (vr(V0 + l * T + j), vr(V0 + j)))
            idx_on(h, "s70", ["SRC0"])
            for j in range(T):
                r = vr(V0 + l * T + j)
                valu(h, "%s %s, %s, %s" % (OPS[op], r, vr(V0 + j), r))
            epilogue(h)
            hs.append(h)
    for op, ins in (("add", "v_add_f32_e32"), ("mul", "v_mul_f32_e32"), ("sub", "v_subrev_f32_e32")):
        for l in range(D):
            h = Handler(K["XC"], OP_ID[op], l)     # push x[a] op c
            prologue(h, const=True, index=["SRC1"])
            for j in range(T):
                valu(h, "%s %s, s72, %s" % (ins, vr(V0 + l * T + j), vr(V0 + j)))
            epilogue(h)
            hs.append(h)
    for l in range(D):
        h = Handler(K["CX"], OP_ID["sub"], l)      # push c - x[b]
        prologue(h, const=True, index=["SRC1"])
        for j in range(T):
            valu(h, "v_sub_f32_e32 %s, s72, %s" % (vr(V0 + l * T + j), vr(V0 + j)))
        epilogue(h)
        hs.append(h)
    for l in range(D):
        h = Handler(K["PUSHX"], 0, l)              # s[l] = x[a] (a lone variable, an operand of IF)
        prologue(h, index=["SRC0"])
        for j in range(T):
            valu(h, "v_mov_b32_e32 %s, %s" % (vr(V0 + l * T + j), vr(V0 + j)))
        epilogue(h)
        hs.append(h)
    h = Handler(K["PUSHC"])                        # s[l] = c; index l*T
    prologue(h, const=True, index=["DST"])
    for j in range(T):
        valu(h, "v_mov_b32_e32 %s, s72" % vr(V0 + j))
    epilogue(h)
    hs.append(h)

    for kind in ("DVV", "DVC", "DCV"):
        hs.append(div_handler(kind, T, V0))
    for op in list(CMP_OPS) + list(LOGIC_OPS):
        for kind in ("CVV", "CVC", "CCV"):
            hs.append(cmp_handler(kind, op, T, V0, ring))
    if not ring:
        hs.append(if_handler(T, V0))
    else:
        ring_handlers(hs, T, D, V0, prologue, epilogue, valu)
        for l in range(D if mode == 4 else 0):
            hs.append(Handler(K["PUSHR"], 0, l))
            hs[-1].row = (V0 + l * T, row_address(V0), V0 - 1, rows_base(T, D, NF, NCV, mode))

    if mode >= 3:                      # trees only: no linear handlers
        return finish(hs, tag, V0, FO, ring, mode)

    # ---------------------------------------------------------------- linear
    R = LIN_REGS
    for op in ("add", "sub", "mul"):
        for d in range(R):
            for s1 in range(R):
                h = Handler(K["RR"], OP_ID[op], d, s1)   # r[d] = r[s1] op src2 (index)
                prologue(h, index=["SRC1"])
                for j in range(T):
                    valu(h, "%s %s, %s, %s" % (OPS[op], vr(V0 + d * T + j), vr(V0 + s1 * T + j), vr(V0 + j)))
                epilogue(h)
                hs.append(h)
    for d in range(R):
        for s2 in range(R):
            h = Handler(K["XR"], OP_ID["sub"], d, s2)    # r[d] = src1 (index) - r[s2]
            prologue(h, index=["SRC0"])
            for j in range(T):
                valu(h, "v_sub_f32_e32 %s, %s, %s" % (vr(V0 + d * T + j), vr(V0 + j), vr(V0 + s2 * T + j)))
            epilogue(h)
            hs.append(h)
    for op in ("add", "sub", "mul"):
        for d in range(R):
            h = Handler(K["FF"], OP_ID[op], d)           # r[d] = src2; r[d] = src1 op r[d]
            prologue(h, second_index=True)
            idx_on(h, "s71", ["SRC0"])
            for j in range(T):
                valu(h, "v_mov_b32_e32 %s, %s" % (vr(V0 + d * T + j), vr(V0 + j)))
            idx_on(h, "s70", ["SRC0"])
            for j in range(T):
                r = vr(V0 + d * T + j)
                valu(h, "%s %s, %s, %s" % (OPS[op], r, vr(V0 + j), r))
            epilogue(h)
            hs.append(h)
    for op in ("add", "sub", "mul"):
        for d in range(R):
            h = Handler(K["CR"], OP_ID[op], d)           # r[d] = c op src (index)
            prologue(h, const=True, index=["SRC1"])
            for j in range(T):
                valu(h, "%s %s, s72, %s" % (OPS[op], vr(V0 + d * T + j), vr(V0 + j)))
            epilogue(h)
            hs.append(h)
    for d in range(R):
        h = Handler(K["RC"], OP_ID["sub"], d)            # r[d] = src (index) - c
        prologue(h, const=True, index=["SRC1"])
        for j in range(T):
            valu(h, "v_subrev_f32_e32 %s, s72, %s" % (vr(V0 + d * T + j), vr(V0 + j)))
        epilogue(h)
        hs.append(h)
    for d in range(R):
        h = Handler(K["MOVC"], 0, d)                     # r[d] = c
        prologue(h, const=True, index="off")
        for j in range(T):
            valu(h, "v_mov_b32_e32 %s, s72" % vr(V0 + d * T + j))
        epilogue(h)
        hs.append(h)
    for d in range(R):
        h = Handler(K["MOVX"], 0, d)                     # r[d] = src (index)
        prologue(h, index=["SRC0"])
        for j in range(T):
            valu(h, "v_mov_b32_e32 %s, %s" % (vr(V0 + d * T + j), vr(V0 + j)))
        epilogue(h)
        hs.append(h)

    return finish(hs, tag, V0, FO, ring, mode)


def ring_handlers(hs, T, D, V0, prologue, epilogue, valu):
    """Classification functions and divisions of a ring core.  Operands on the
    stack lie next to each other (or at a level the handler knows), so one
    index serves a whole instruction: a compare and a select a slot, where the
    general form also copies an operand and sets three indexes a slot.  Masks
    go to s[64:71], four slots at a time, which also spaces a compare from
    the select that reads it."""
    def masked(h, test, d, sel):
        for j0 in range(0, T, 4):
            for j in range(j0, j0 + 4):
                test(h, j, "s[%d:%d]" % (64 + 2 * (j - j0), 65 + 2 * (j - j0)))
            for j in range(j0, j0 + 4):
                valu(h, "v_cndmask_b32_e64 %s, %s, s[%d:%d]" % (d(j), sel(j), 64 + 2 * (j - j0), 65 + 2 * (j - j0)))

    def tester(op, a, b):
        """mask = a(j) op b(j)"""
        def test(h, j, m):
            if op in CMP_OPS:
                valu(h, "v_cmp_%s_f32_e64 %s, %s, %s" % (CMP_OPS[op], m, a(j), b(j)))
            else:
                valu(h, "v_cmp_neq_f32_e64 %s, 0, %s" % (m, a(j)))
                valu(h, "v_cmp_neq_f32_e32 vcc, 0, %s" % b(j))
                h.emit("%s %s, vcc, %s" % (LOGIC_OPS[op], m, m), 4)
        return test

    for op in list(CMP_OPS) + list(LOGIC_OPS):
        h = Handler(K["CSS"], op)                   # s[h-2] = s[h-2] op s[h-1]; index (h-2)*T
        prologue(h, index=["SRC0", "SRC1", "DST"])
        masked(h, tester(op, lambda j: vr(V0 + j), lambda j: vr(V0 + T + j)), lambda j: vr(V0 + j), lambda j: "0, 1.0")
        epilogue(h)
        hs.append(h)
        for l in range(D):
            h = Handler(K["CSX"], op, l)            # s[l] = s[l] op x; index = feature offset
            lev = lambda j, l=l: vr(V0 + l * T + j)   # noqa: E731
            # compares read the variable as their second source, under its index; a test against 0 has the
            # stack entry there, so it goes first, with the index off
            if op in CMP_OPS:
                prologue(h, index=["SRC1"])
                masked(h, tester(op, lev, lambda j: vr(V0 + j)), lev, lambda j: "0, 1.0")
            else:
                prologue(h, index=["SRC0"])
                swap = lambda h, j, m, op=op, lev=lev: (   # noqa: E731
                    valu(h, "v_cmp_neq_f32_e64 %s, 0, %s" % (m, lev(j))),
                    valu(h, "v_cmp_neq_f32_e64 vcc, %s, 0" % vr(V0 + j)),
                    h.emit("%s %s, vcc, %s" % (LOGIC_OPS[op], m, m), 4))
                masked(h, swap, lev, lambda j: "0, 1.0")
            epilogue(h)
            hs.append(h)
    for pa in range(3):                             # IF of three stack entries, by where each operand landed
        for pb in range(3):
            if pa == pb:
                continue
            pc = 3 - pa - pb
            h = Handler(K["IF3"], 15, 3 * pa + pb)
            prologue(h, index=["SRC0", "SRC1", "DST"])
            masked(h, lambda h, j, m: valu(h, "v_cmp_neq_f32_e64 %s, 0, %s" % (m, vr(V0 + pa * T + j))),
                   lambda j: vr(V0 + j), lambda j: "%s, %s" % (vr(V0 + pc * T + j), vr(V0 + pb * T + j)))
            epilogue(h)
            hs.append(h)
    # divisions: the arithmetic itself is shared by the phases (division_bodies)
    for l in range(D - 1):
        for kind in ("DSS", "DSSR", "DSX", "DXS"):
            h = Handler(K[kind], 3, l)
            if kind in ("DSX", "DXS"):              # the variable is copied to the level above
                prologue(h, index=["SRC0"])
                for j in range(T):
                    valu(h, "v_mov_b32_e32 %s, %s" % (vr(V0 + (l + 1) * T + j), vr(V0 + j)))
                h.emit("s_set_gpr_idx_off", 4)
            else:
                prologue(h, index="off")
            h.then = "%s%d" % ("dss" if kind in ("DSS", "DSX") else "dssr", l)
            epilogue(h)
            hs.append(h)


def division_bodies(T, D, V0, tag):
    """s[l] = s[l] / s[l+1] (dss) or s[l+1] / s[l] (dssr), protected; on to the address in s[76:77].  The sequence of
    div_handler without copies: the test of the divisor goes first, to s[64:65]."""
    tD, tR, tN, tE, tF = (vr(V0 - DIV_TMP + k) for k in range(2, 7))
    L = []
    for l in range(D - 1):
        for name in ("dss", "dssr"):
            L += [".Lgpx_%s%d_%s:" % (name, l, tag), "s_mov_b32 s80, 0x%x" % DIV_THRESHOLD]
            for j in range(T):
                d = vr(V0 + l * T + j)
                A, B = (d, vr(V0 + (l + 1) * T + j)) if name == "dss" else (vr(V0 + (l + 1) * T + j), d)
                L += ["v_div_scale_f32 %s, vcc, %s, %s, %s" % (tD, B, B, A),
                      "v_cmp_nlt_f32_e64 s[64:65], |%s|, s80" % B,
                      "v_rcp_f32_e32 %s, %s" % (tR, tD),
                      "v_div_scale_f32 %s, vcc, %s, %s, %s" % (tN, A, B, A),
                      "v_fma_f32 %s, -%s, %s, 1.0" % (tE, tD, tR),
                      "v_fmac_f32_e32 %s, %s, %s" % (tR, tE, tR),
                      "v_mul_f32_e32 %s, %s, %s" % (tE, tN, tR),
                      "v_fma_f32 %s, -%s, %s, %s" % (tF, tD, tE, tN),
                      "v_fmac_f32_e32 %s, %s, %s" % (tE, tF, tR),
                      "v_fma_f32 %s, -%s, %s, %s" % (tD, tD, tE, tN),
                      "v_div_fmas_f32 %s, %s, %s, %s" % (tD, tD, tR, tE),
                      "v_div_fixup_f32 %s, %s, %s, %s" % (tD, tD, B, A),
                      "v_cndmask_b32_e64 %s, 1.0, %s, s[64:65]" % (d, tD)]
            L += ["s_setpc_b64 s[76:77]"]
    return L


def div_handler(kind, T, V0):
    """Protected division in the core: d = |b| < 1e-6f ? 1 : a / b for the
    T slots, a and b at offsets (or the constant), d at a third offset, all
    in the exit's payload layout (byte 0 a, byte 1 b, byte 2 d).

    The quotient is the correctly rounded IEEE one, by the sequence the
    compiler emits for a binary32 division with denormals kept: scale
    operands (v_div_scale), reciprocal, two Newton-Raphson refinements of it
    and of the quotient with fused multiply-adds, the scaled fused add
    (v_div_fmas, whose scale flag is vcc) and the special-case fix-up
    (v_div_fixup).  Its dependent reads keep the compiler's spacing: one
    instruction between the reciprocal and its first use, six between the
    vcc write and v_div_fmas, two wait states between the compare's vcc
    write and the select that reads it.  Operands are copied out of the index range
    slot by slot (the index mode offsets every VGPR of the enabled fields,
    so the arithmetic runs with it off), and the select writes the result
    through the destination index."""
    a_const, b_const = kind == "DCV", kind == "DVC"
    tA, tB, tD, tR, tN, tE, tF = (vr(V0 - DIV_TMP + k) for k in range(DIV_TMP))

    def body(A, B, Dx, C):
        L = ["s_mov_b32 s80, 0x%x" % DIV_THRESHOLD]
        if a_const or b_const:
            L.append("s_set_gpr_idx_off")
            L.append("v_mov_b32_e32 %s, %s" % (tA if a_const else tB, C))
        for j in range(T):
            if not a_const:
                L.append("s_set_gpr_idx_on %s, gpr_idx(SRC0)" % A)
                L.append("v_mov_b32_e32 %s, %s" % (tA, vr(V0 + j)))
            if not b_const:
                L.append("s_set_gpr_idx_on %s, gpr_idx(SRC0)" % B)
                L.append("v_mov_b32_e32 %s, %s" % (tB, vr(V0 + j)))
            L.append("s_set_gpr_idx_off")
            L += ["v_div_scale_f32 %s, vcc, %s, %s, %s" % (tD, tB, tB, tA),
                  "v_rcp_f32_e32 %s, %s" % (tR, tD),
                  "v_div_scale_f32 %s, vcc, %s, %s, %s" % (tN, tA, tB, tA),
                  "v_fma_f32 %s, -%s, %s, 1.0" % (tE, tD, tR),
                  "v_fmac_f32_e32 %s, %s, %s" % (tR, tE, tR),
                  "v_mul_f32_e32 %s, %s, %s" % (tE, tN, tR),
                  "v_fma_f32 %s, -%s, %s, %s" % (tF, tD, tE, tN),
                  "v_fmac_f32_e32 %s, %s, %s" % (tE, tF, tR),
                  "v_fma_f32 %s, -%s, %s, %s" % (tD, tD, tE, tN),
                  "v_div_fmas_f32 %s, %s, %s, %s" % (tD, tD, tR, tE),
                  "v_div_fixup_f32 %s, %s, %s, %s" % (tD, tD, tB, tA),
                  # vcc = |b| >= 1e-6f or b is NaN: keep the quotient, else 1
                  "v_cmp_nlt_f32_e64 vcc, |%s|, s80" % tB,
                  # a vector write of a mask register is read as a lane mask two wait states later at the earliest
                  "s_nop 1",
                  "s_set_gpr_idx_on %s, gpr_idx(DST)" % Dx,
                  "v_cndmask_b32_e32 %s, 1.0, %s, vcc" % (vr(V0 + j), tD)]
        return L

    h = Handler(K[kind], 3)
    # phase A: own record in s[64:67], the next one already in s[68:71]
    la = ["s_lshr_b32 s74, s66, 8", "s_lshr_b32 s79, s66, 16"] + body("s66", "s74", "s79", "s67")
    la += ["s_add_u32 s62, s62, 16", "s_setpc_b64 s[68:69]"]
    # phase B: own record in s[68:71], saved before the load of the next two
    lb = ["s_mov_b32 s73, s70", "s_lshr_b32 s74, s70, 8", "s_lshr_b32 s79, s70, 16", "s_mov_b32 s72, s71",
          "s_add_u32 s62, s62, 16", "s_load_dwordx8 s[64:71], s[60:61], s62"] + body("s73", "s74", "s79", "s72")
    lb += ["s_waitcnt lgkmcnt(0)", "s_setpc_b64 s[64:65]"]
    h.phases, h.body, h.n_idx = (la, lb), lambda A, B, Dx, C, _: body(A, B, Dx, C), 3
    return h


# The classification functions in the core: >, <, == give 1 or 0 (an ordered
# compare: false with a NaN); AND and OR test operands for != 0 (a NaN is
# non-zero); IF(a, b, c) = a != 0 ? b : c.  Operand ids as the tree opcodes.
CMP_OPS = {12: "gt", 13: "lt", 14: "eq"}
CMP_SWAP = {"gt": "lt", "lt": "gt", "eq": "eq"}      # c op x  ==  x swap(op) c
LOGIC_OPS = {8: "s_and_b64", 9: "s_or_b64"}
IF_KIND = "IF3"


def phases_of(h, body, n_idx):
    """Both phases of a handler whose body takes its index registers (A, B,
    D[, C]) and the constant register.  Phase A finds its record in s[64:67]
    (the next one is already in s[68:71]); phase B saves what it needs from
    s[68:71] before loading the next two records over s[64:71]."""
    if n_idx == 3:
        la = ["s_lshr_b32 s74, s66, 8", "s_lshr_b32 s79, s66, 16"] + body("s66", "s74", "s79", "s67", None)
        lb = ["s_mov_b32 s73, s70", "s_lshr_b32 s74, s70, 8", "s_lshr_b32 s79, s70, 16", "s_mov_b32 s72, s71"]
        regs_b = ("s73", "s74", "s79", "s72", None)
    else:
        la = ["s_lshr_b32 s74, s66, 8", "s_lshr_b32 s73, s66, 16", "s_lshr_b32 s79, s66, 24"] + \
            body("s66", "s74", "s79", None, "s73")
        lb = ["s_mov_b32 s73, s70", "s_lshr_b32 s74, s70, 8", "s_lshr_b32 s72, s70, 16", "s_lshr_b32 s79, s70, 24"]
        regs_b = ("s73", "s74", "s79", None, "s72")
    la += ["s_add_u32 s62, s62, 16", "s_setpc_b64 s[68:69]"]
    lb += ["s_add_u32 s62, s62, 16", "s_load_dwordx8 s[64:71], s[60:61], s62"] + body(*regs_b)
    lb += ["s_waitcnt lgkmcnt(0)", "s_setpc_b64 s[64:65]"]
    h.phases, h.body, h.n_idx = (la, lb), body, n_idx
    return h


def cmp_handler(kind, op, T, V0, ring=False):
    """d = a op b for op in >, <, ==, AND, OR (1 or 0 per slot), a and b at
    two offsets (CVV) or one of them the record's constant (CVC: b, CCV: a),
    d at a third; the payload is the exit's layout.  A compare writes vcc
    (AND and OR first write the first operand's test to s[80:81] and combine
    them); a select through the destination index writes the result, two wait
    states after the mask is written."""
    a_const, b_const = kind == "CCV", kind == "CVC"
    tB = vr(V0 - DIV_TMP)
    name = CMP_OPS.get(op)

    def body(A, B, Dx, C, _):
        L = []
        if name is None and (a_const or b_const):
            # the constant's truth is the same in every lane
            L += ["v_cmp_neq_f32_e64 s[80:81], 0, %s" % C]
        for j in range(T):
            if name is not None:
                if a_const:          # c op b
                    L += ["s_set_gpr_idx_on %s, gpr_idx(SRC1)" % B,
                          "v_cmp_%s_f32_e32 vcc, %s, %s" % (name, C, vr(V0 + j))]
                elif b_const:        # a op c  ==  c swap(op) a
                    L += ["s_set_gpr_idx_on %s, gpr_idx(SRC1)" % A,
                          "v_cmp_%s_f32_e32 vcc, %s, %s" % (CMP_SWAP[name], C, vr(V0 + j))]
                else:                # b copied out, a through the index
                    L += ["s_set_gpr_idx_on %s, gpr_idx(SRC0)" % B,
                          "v_mov_b32_e32 %s, %s" % (tB, vr(V0 + j)),
                          "s_set_gpr_idx_on %s, gpr_idx(SRC0)" % A,
                          "v_cmp_%s_f32_e32 vcc, %s, %s" % (name, vr(V0 + j), tB)]
            else:
                if not (a_const or b_const):
                    L += ["s_set_gpr_idx_on %s, gpr_idx(SRC1)" % A,
                          "v_cmp_neq_f32_e64 s[80:81], 0, %s" % vr(V0 + j)]
                L += ["s_set_gpr_idx_on %s, gpr_idx(SRC1)" % (A if b_const else B),
                      "v_cmp_neq_f32_e32 vcc, 0, %s" % vr(V0 + j),
                      "s_nop 1",
                      "%s vcc, vcc, s[80:81]" % LOGIC_OPS[op]]
            L += ["s_nop 1",
                  "s_set_gpr_idx_on %s, gpr_idx(DST)" % Dx,
                  "v_cndmask_b32_e64 %s, 0, 1.0, vcc" % vr(V0 + j)]
        return L

    def body_by_four(A, B, Dx, C, _):
        """Ring cores: the same four slots at a time, masks in s[64:71], one index for each pass."""
        L = []
        if name is None and (a_const or b_const):
            L += ["v_cmp_neq_f32_e64 s[80:81], 0, %s" % C]
        for j0 in range(0, T, 4):
            js = range(j0, j0 + 4)
            m = {j: "s[%d:%d]" % (64 + 2 * (j - j0), 65 + 2 * (j - j0)) for j in js}
            t = {j: vr(V0 - DIV_TMP + j - j0) for j in js}
            first = B if a_const or (name is not None and not b_const) else A
            if name is not None and not (a_const or b_const):
                L += ["s_set_gpr_idx_on %s, gpr_idx(SRC0)" % B] + ["v_mov_b32_e32 %s, %s" % (t[j], vr(V0 + j)) for j in js]
                L += ["s_set_gpr_idx_on %s, gpr_idx(SRC0)" % A]
                L += ["v_cmp_%s_f32_e64 %s, %s, %s" % (name, m[j], vr(V0 + j), t[j]) for j in js]
            elif name is not None:
                rel = name if a_const else CMP_SWAP[name]
                L += ["s_set_gpr_idx_on %s, gpr_idx(SRC1)" % first]
                L += ["v_cmp_%s_f32_e64 %s, %s, %s" % (rel, m[j], C, vr(V0 + j)) for j in js]
            else:
                L += ["s_set_gpr_idx_on %s, gpr_idx(SRC1)" % first]
                L += ["v_cmp_neq_f32_e64 %s, 0, %s" % (m[j], vr(V0 + j)) for j in js]
                if not (a_const or b_const):
                    L += ["s_set_gpr_idx_on %s, gpr_idx(SRC1)" % B]
                for j in js:
                    if not (a_const or b_const):
                        L += ["v_cmp_neq_f32_e32 vcc, 0, %s" % vr(V0 + j)]
                    L += ["%s %s, %s, %s" % (LOGIC_OPS[op], m[j], "s[80:81]" if a_const or b_const else "vcc", m[j])]
            L += ["s_set_gpr_idx_on %s, gpr_idx(DST)" % Dx]
            L += ["v_cndmask_b32_e64 %s, 0, 1.0, %s" % (vr(V0 + j), m[j]) for j in js]
        return L

    if ring:
        h = Handler(K[kind], op)
        h.body, h.n_idx = body_by_four, 3
        return h
    return phases_of(Handler(K[kind], op), body, 3)


def if_handler(T, V0):
    """IF(a, b, c) = a != 0 ? b : c (a NaN is non-zero) over three offsets,
    the result to a fourth (payload bytes 0-3: a, b, c, d)."""
    tB, tC = vr(V0 - DIV_TMP), vr(V0 - DIV_TMP + 1)

    def body(A, B, Dx, _, Cx):
        L = []
        for j in range(T):
            L += ["s_set_gpr_idx_on %s, gpr_idx(SRC0)" % B,
                  "v_mov_b32_e32 %s, %s" % (tB, vr(V0 + j)),
                  "s_set_gpr_idx_on %s, gpr_idx(SRC0)" % Cx,
                  "v_mov_b32_e32 %s, %s" % (tC, vr(V0 + j)),
                  "s_set_gpr_idx_on %s, gpr_idx(SRC1)" % A,
                  "v_cmp_neq_f32_e32 vcc, 0, %s" % vr(V0 + j),
                  "s_nop 1",
                  "s_set_gpr_idx_on %s, gpr_idx(DST)" % Dx,
                  "v_cndmask_b32_e32 %s, %s, %s, vcc" % (vr(V0 + j), tC, tB)]
        return L

    return phases_of(Handler(K[IF_KIND], 15), body, 4)


def bool_handlers(hs, T, D, V0, FO, prologue, idx_on, epilogue, valu):
    """Handlers of the Boolean function set.  Every function is symmetric, so
    only the forms with the stack (or first) operand on the left exist: SS,
    SX, XX2 (two features, two passes) and PUSHX.  Each function is one
    vector instruction per slot; the index mode offsets the same sources and
    destination in every encoding."""
    for op in BOOL_OPS:
        h = Handler(K["SS"], BOOL_ID[op])           # s[h-2] = s[h-2] op s[h-1]; index (h-2)*T
        prologue(h, index=["SRC0", "SRC1", "DST"])
        for j in range(T):
            valu(h, bool_op(op, vr(V0 + j), vr(V0 + j), vr(V0 + T + j)))
        epilogue(h)
        hs.append(h)
    for op in BOOL_OPS:
        for l in range(D):
            h = Handler(K["SX"], BOOL_ID[op], l)    # s[l] = s[l] op x[b]; index = feature offset
            prologue(h, index=["SRC1"])
            for j in range(T):
                r = vr(V0 + l * T + j)
                valu(h, bool_op(op, r, r, vr(V0 + j)))
            epilogue(h)
            hs.append(h)
    for op in BOOL_OPS:
        for l in range(D):
            h = Handler(K["XX2"], BOOL_ID[op], l)   # s[l] = x[b]; s[l] = x[a] op s[l]
            prologue(h, second_index=True)
            idx_on(h, "s71", ["SRC0"])
            for j in range(T):
                valu(h, "v_mov_b32_e32 %s, %s" % (vr(V0 + l * T + j), vr(V0 + j)))
            idx_on(h, "s70", ["SRC0"])
            for j in range(T):
                r = vr(V0 + l * T + j)
                valu(h, bool_op(op, r, vr(V0 + j), r))
            epilogue(h)
            hs.append(h)
    h = Handler(K["PUSHX"])                         # s[0] = x[a] (a program that is one variable)
    prologue(h, index=["SRC0"])
    for j in range(T):
        valu(h, "v_mov_b32_e32 %s, %s" % (vr(V0 + j), vr(V0 + j)))
    epilogue(h)
    hs.append(h)


def finish(hs, tag, V0, FO, ring=False, mode=0):
    """Every phase of every handler (two, or four in a ring core), laid out in slots."""
    if ring:
        # all phases of the plain arithmetic first, so that they lie close together in the instruction cache
        plain = [h for h in hs if h.kind < K["DVV"]]
        rest = [h for h in hs if h.kind >= K["DVV"]]
        hs, unit = [phase_ring(h, k, tag, ring_base(mode)) for g in (plain, rest) for k in range(4) for h in g], RING_SLOT
    else:
        hs, unit = [phase_a(h, tag) for h in hs] + [phase_b(h, tag) for h in hs], SLOT
    slot = 0
    for h in hs:
        h.slot = slot
        slot += (h.size + unit - 1) // unit
    return tag, V0, FO, hs, slot


# Ring cores.  The pair scheme below still waits once in two instructions for
# most of the scalar cache's latency (measured on the 20-multiplexer: 43 of
# the 100 cycles an instruction takes a wave).  A ring core keeps four records,
# two pairs, in 16 scalar registers and has four phases of every handler: phase k works
# from record k and jumps to record k + 1.  The odd phases first wait for the
# other pair, requested two instructions ago, then, their own pair being used
# up, request the pair after it.  s62 is the byte offset of the pair requested
# last: the record after an exit is at s62 - 16 in an even phase, at s62 in an
# odd one.  Twice the handlers, so the slots are 32 bytes.
RING_SLOT = 32
RING_PHASE = 6                   # the phase's place in a handler key's kind


def ring_base(mode):
    """First register of the ring: beside the series coefficients where there are any."""
    return 8 if mode == 4 else 36


def phase_ring(h, k, tag, base):
    c = _copy(h, h.kind | (k << RING_PHASE))
    r = base + 4 * k
    pay, cst = "s%d" % (r + 2), "s%d" % (r + 3)
    own = base + 8 * (k >> 1)
    nxt = "s_setpc_b64 %s" % sp(base + 4 * ((k + 1) & 3))
    odd = k & 1
    fetch = ["s_add_u32 s62, s62, 32", "s_load_dwordx8 s[%d:%d], s[60:61], s62" % (own, own + 7)]
    if h.kind == K["EXIT"]:
        L = ["s_set_gpr_idx_off"] + ([] if odd else ["s_sub_u32 s62, s62, 16"]) + \
            ["s_mov_b32 s66, %s" % pay, "s_mov_b32 s67, %s" % cst, "s_branch .Lgpx_end_%s" % tag]
    elif h.row:
        # the pair is requested after the row has come, so that only the row is waited for
        reg, at, tmp, base_lds = h.row
        L = ["s_waitcnt lgkmcnt(0)"] if odd else []
        L += ["s_set_gpr_idx_off", "v_add_u32_e32 v%d, %s, v%d" % (tmp, pay, at),
              "ds_read_b128 %s, v%d offset:%d" % (quad(reg), tmp, base_lds), "s_waitcnt lgkmcnt(0)"]
        L += (fetch if odd else []) + [nxt]
    elif h.body and not odd:
        if h.n_idx == 3:
            L = ["s_lshr_b32 s74, %s, 8" % pay, "s_lshr_b32 s79, %s, 16" % pay] + h.body(pay, "s74", "s79", cst, None)
        else:
            L = ["s_lshr_b32 s74, %s, 8" % pay, "s_lshr_b32 s73, %s, 16" % pay, "s_lshr_b32 s79, %s, 24" % pay] + \
                h.body(pay, "s74", "s79", None, "s73")
        L += [nxt]
    elif h.body:
        L = ["s_waitcnt lgkmcnt(0)", "s_mov_b32 s73, %s" % pay, "s_lshr_b32 s74, %s, 8" % pay]
        if h.n_idx == 3:
            L += ["s_lshr_b32 s79, %s, 16" % pay, "s_mov_b32 s72, %s" % cst] + fetch + h.body("s73", "s74", "s79", "s72", None)
        else:
            L += ["s_lshr_b32 s72, %s, 16" % pay, "s_lshr_b32 s79, %s, 24" % pay] + fetch + \
                h.body("s73", "s74", "s79", None, "s72")
        L += [nxt]
    else:
        L = ["s_waitcnt lgkmcnt(0)"] if odd else []
        for x in h.lines:
            if x.startswith(("s_waitcnt", "s_setpc")):
                continue
            if x == "s_mov_b32 s72, s67":
                if odd:
                    L.append("s_mov_b32 s72, %s" % cst)
            elif x == "s_mov_b32 s70, s66":
                if odd:
                    L.append("s_mov_b32 s73, %s" % pay)
            elif x == "s_lshr_b32 s71, s66, 8":
                L.append("s_lshr_b32 s74, %s, 8" % pay)
            elif x.startswith("s_add_u32 s62"):
                if odd:
                    L += fetch
            elif x.startswith("s_load_dwordx4"):
                pass
            else:
                x = x.replace("s_set_gpr_idx_on s66,", "s_set_gpr_idx_on %s," % pay)
                x = x.replace("s_set_gpr_idx_on s70,", "s_set_gpr_idx_on %s," % ("s73" if odd else pay))
                x = x.replace("s_set_gpr_idx_on s71,", "s_set_gpr_idx_on s74,")
                L.append(x if odd else x.replace("s72", cst))
        if h.then:
            L += ["s_mov_b64 s[76:77], %s" % sp(base + 4 * ((k + 1) & 3)), "s_branch .Lgpx_%s_%s" % (h.then, tag)]
        else:
            L += [nxt]
    for x in L:
        c.emit(x, insn_bytes(x))
    return c


# Two copies of every handler.  Records are fetched two at a time: a phase-B
# handler (its own record in s[68:71]) loads the next two records into
# s[64:71] with one s_load_dwordx8, works, waits, and jumps to the next
# instruction's phase-A handler; a phase-A handler (its record in s[64:67],
# the next one already in s[68:71]) works and jumps on without loading or
# waiting.  So only every second instruction waits for the scalar cache.
# The host gives instructions alternating phases, A first after every entry
# into the core (program start, return from an exit), which loads the first
# two records itself.  The handlers are written once (as for a single record
# in s[64:67], constant copied to s72, indexes in s66/s70/s71); these
# functions rewrite them for each phase.
PHASE_B = 0x80


def _copy(h, kind):
    c = Handler(kind, h.op, h.p1, h.p2)
    return c


def phase_a(h, tag):
    c = _copy(h, h.kind)
    if h.phases:
        for x in h.phases[0]:
            c.emit(x, insn_bytes(x))
        return c
    if h.kind == K["EXIT"]:
        for x in h.lines:
            c.emit(x, 4)
        return c
    body = []
    for x in h.lines:
        if x == "s_mov_b32 s72, s67" or x == "s_mov_b32 s70, s66" or x.startswith("s_add_u32 s62") \
                or x.startswith("s_load_dwordx4") or x.startswith("s_waitcnt") or x.startswith("s_setpc"):
            continue
        x = x.replace("s_lshr_b32 s71, s66, 8", "s_lshr_b32 s74, s66, 8")
        x = x.replace("s_set_gpr_idx_on s70,", "s_set_gpr_idx_on s66,").replace("s_set_gpr_idx_on s71,", "s_set_gpr_idx_on s74,")
        x = x.replace("s72", "s67")
        body.append(x)
    for x in body:
        c.emit(x, insn_bytes(x))
    c.emit("s_add_u32 s62, s62, 16", 4)
    c.emit("s_setpc_b64 s[68:69]", 4)
    return c


def phase_b(h, tag):
    c = _copy(h, h.kind | PHASE_B)
    if h.phases:
        for x in h.phases[1]:
            c.emit(x, insn_bytes(x))
        return c
    if h.kind == K["EXIT"]:
        c.emit("s_set_gpr_idx_off", 4)
        c.emit("s_mov_b32 s66, s70", 4)
        c.emit("s_mov_b32 s67, s71", 4)
        c.emit("s_branch .Lgpx_end_%s" % tag, 4)
        return c
    for x in h.lines:
        if x == "s_mov_b32 s72, s67":
            x = "s_mov_b32 s72, s71"
        elif x == "s_mov_b32 s70, s66":
            x = "s_mov_b32 s73, s70"
        elif x == "s_lshr_b32 s71, s66, 8":
            x = "s_lshr_b32 s74, s70, 8"
        elif x.startswith("s_load_dwordx4"):
            x = "s_load_dwordx8 s[64:71], s[60:61], s62"
        elif x.startswith("s_set_gpr_idx_on s66,"):
            x = x.replace("s_set_gpr_idx_on s66,", "s_set_gpr_idx_on s70,")
        elif x.startswith("s_set_gpr_idx_on s70,"):
            x = x.replace("s_set_gpr_idx_on s70,", "s_set_gpr_idx_on s73,")
        elif x.startswith("s_set_gpr_idx_on s71,"):
            x = x.replace("s_set_gpr_idx_on s71,", "s_set_gpr_idx_on s74,")
        c.emit(x, insn_bytes(x))
    return c


# ---------------------------------------------------------------------------
# Around the handlers: the unit's tile, the end of a program, sin/cos/exp/log
# ---------------------------------------------------------------------------
# Scalar registers the block is entered with (besides s[60:62], s63, s78):
#   s[82:83] case matrix at the tile's first case   s[84:85] bytes from one feature row to the next
#   s86 features to load    s87 cases from the tile's start to the end of the data (at most the tile)
#   s[88:89] targets at the tile                    s[90:91] partial sums of the tile's first block
#   s92 bytes from one program's partial sums to the next
#   s93 fitness kind        s[94:95] per-case outputs at the tile    s96 byte offset where the unit's code ends
#   s97 LDS address of the wave's targets           s98 bits from the tile's start to the end (Boolean)
#   s[100:101] the series coefficients (COEF)
# Ring cores with sin/cos/exp/log first run the programs that compute their share of the tile's rows (kind TO_ROW),
# meet the block's other waves, and go on to their own:
#   s56, s57 byte offsets of those, s98 their kind; s98 = -1: no rows, s62, s96 and s93 are the wave's own
# s[24:55] hold the coefficients (kernels with sin/cos/exp/log); s58, s59, s79-s81, s99, s72-s77 are temporaries.
PF_LINES = 14                    # 64-byte lines of the next program fetched beside its first records
FIT_SUM_ABS, FIT_MSE, FIT_HITS, OUT_CASES, FIT_CLASS, TO_ROW = 0, 1, 2, 3, 4, 5

# binary64 series constants in SGPR pairs, in the order of gmath::kCoreCoef
COEF = {n: 24 + 2 * i for i, n in enumerate(
    ("KPI", "P1", "P2", "P3", "S0", "S2", "C2", "KLN", "L1", "L2", "E1", "E3", "LN2", "G1", "G2", "G4"))}
# constants a VOP3 needs in VGPRs beside one of those (it reads one scalar pair): high and low words
VCONST = {"R": (0x43380000, 0x00000000), "S1": (0x3F811111, 0x11111111), "C1": (0x3FA55555, 0x55555555),
          "E2": (0x3FA55555, 0x55555555), "G3": (0x3FC99999, 0x9999999A)}
# LDS byte offsets of the reduction tables (gp_math.h: kTabSC, kTabExp, kTabLog, kTabPi, in doubles)
LDS_SC, LDS_EXP, LDS_LOG = 0, 256 * 8, 320 * 8
LDS_PI = LDS_LOG + 2 * 257 * 8
LOG_K0 = 0x7E6A


def transc_slots(NCV):
    """Slots whose sin/cos/exp/log are computed side by side: two where the compiler's range has room."""
    return 2 if NCV >= 48 else 1


def work_regs(NCV, mode, ring=False):
    """VGPRs below the core's range that the block uses (and clobbers)."""
    if mode in (0, 4):
        n = 14 * transc_slots(NCV) + 2 + (2 if ring and mode == 4 else 0)    # a lane's offset in a row, alone at the bottom
        return n + (2 * len(VCONST) if NCV >= 64 else 0)
    return 0 if mode == 2 else DIV_TMP


def pair(n):
    return "v[%d:%d]" % (n, n + 1)


def quad(n):
    return "v[%d:%d]" % (n, n + 3)


def sp(n):
    return "s[%d:%d]" % (n, n + 1)


def exec_slot(j, left="s87"):
    """exec = the lanes of slot j that hold a case: 64 j + lane < left."""
    return ["s_sub_i32 s72, %s, %d" % (left, 64 * j),
            "s_bfm_b64 s[74:75], s72, 0",
            "s_cmp_gt_i32 s72, 63",
            "s_cselect_b64 s[74:75], -1, s[74:75]",
            "s_cmp_lt_i32 s72, 1",
            "s_cselect_b64 exec, 0, s[74:75]"]


def first_records(ring, mode=0):
    """Requests the records at s62, and enters the program there once they have come."""
    if ring:
        b = ring_base(mode)
        return "s_load_dwordx16 s[%d:%d], s[60:61], s62" % (b, b + 15), \
            ["s_add_u32 s62, s62, 32", "s_setpc_b64 %s" % sp(b)]
    return "s_load_dwordx8 s[64:71], s[60:61], s62", ["s_setpc_b64 s[64:65]"]


def unit_start(T, D, NF, V0, FO, tag, mode, ring):
    """Start of a unit: the first records and code lines (into the scalar
    cache), the tile's targets (to LDS, read again at the end of every
    program) and features (straight into their registers), all in flight
    together.  Rows of lanes past the data are not read."""
    vl4, vy = "v%d" % (V0 + T), "v%d" % (V0 + T + 1)     # stack level 1 is free here
    L = ["v_mbcnt_lo_u32_b32 %s, -1, 0" % vy, "v_mbcnt_hi_u32_b32 %s, -1, %s" % (vy, vy),
         "v_lshlrev_b32_e32 %s, 2, %s" % (vl4, vy), "v_lshl_add_u32 %s, %s, 4, s97" % (vy, vy),
         first_records(ring, mode)[0]]
    rows = ring and mode == 4
    if rows:
        # the block's rows are no longer read when every wave is here
        L += ["v_lshlrev_b32_e32 v%d, 2, %s" % (row_address(V0), vl4),
              "s_cmp_eq_u32 s98, -1", "s_cbranch_scc1 .Lgpx_alone_%s" % tag, "s_barrier", ".Lgpx_alone_%s:" % tag]
    if mode in (0, 4):
        L += ["s_load_dwordx16 s[24:39], s[100:101], 0x0", "s_load_dwordx16 s[40:55], s[100:101], 0x40"]
    L += prefetch_start(tag, "0", "s96") + ["s_mov_b32 s99, 0"]
    for j in range(T):
        L += exec_slot(j)
        L += ["s_cbranch_execz .Lgpx_tile_%s" % tag]
        L += ["s_cmp_eq_u32 s93, %d" % OUT_CASES, "s_cbranch_scc1 .Lgpx_noy%d_%s" % (j, tag),
              "global_load_dword v%d, %s, s[88:89] offset:%d" % (V0 + j, vl4, 256 * j),
              ".Lgpx_noy%d_%s:" % (j, tag), "s_mov_b64 s[72:73], s[82:83]"]
        for f in range(NF):
            L += ["s_cmp_le_u32 s86, %d" % f, "s_cbranch_scc1 .Lgpx_row%d_%s" % (j, tag),
                  "global_load_dword v%d, %s, s[72:73] offset:%d" % (V0 + FO + f * T + j, vl4, 256 * j),
                  "s_add_u32 s72, s72, s84", "s_addc_u32 s73, s73, s85"]
        L += [".Lgpx_row%d_%s:" % (j, tag)]
    L += [".Lgpx_tile_%s:" % tag, "s_mov_b64 exec, -1", "s_waitcnt vmcnt(0) lgkmcnt(0)"]
    for k in range(T // 4):
        L += ["ds_write_b128 %s, %s offset:%d" % (vy, quad(V0 + 4 * k), 1024 * k)]
    if mode in (0, 4) and V0 >= 64:
        for i, (hi, lo) in enumerate(VCONST.values()):
            r = vconst_reg(V0, mode, i)
            L += ["v_mov_b32_e32 v%d, 0x%x" % (r, lo), "v_mov_b32_e32 v%d, 0x%x" % (r + 1, hi)]
    L += ["s_waitcnt lgkmcnt(0)", "s_branch .Lgpx_%s_%s" % ("next" if rows else "rest", tag)]
    return L


def vconst_reg(V0, mode, i):
    return V0 - 14 * transc_slots(V0) - 2 - 2 * len(VCONST) + 2 * i


def prefetch_start(tag, n, limit):
    """Fetch the 64-byte lines after the one at s62, up to byte offset
    `limit`, into the scalar cache: at most s78 (<= PF_LINES) now, without
    waiting; s[58:59] and s99 (lines still to fetch) let `rest` go on."""
    L = ["s_and_b32 s72, s62, 0xffffffc0", "s_add_u32 s58, s60, s72", "s_addc_u32 s59, s61, 0",
         "s_sub_u32 s73, %s, 1" % limit, "s_lshr_b32 s73, s73, 6", "s_lshr_b32 s72, s72, 6",
         "s_sub_i32 s99, s73, s72", "s_max_i32 s99, s99, 0", "s_cmp_eq_u32 s78, 0", "s_cselect_b32 s99, 0, s99"]
    return L + prefetch_lines(tag, n)


def prefetch_lines(tag, n):
    """One round: the next min(s99, s78) lines after s[58:59], by a jump into straight-line loads."""
    L = ["s_min_u32 s72, s99, s78", "s_sub_u32 s99, s99, s72",
         "s_lshl_b32 s73, s72, 3", "s_getpc_b64 s[74:75]", ".Lgpx_pf%s_%s:" % (n, tag),
         "s_add_u32 s74, s74, .Lgpx_pfe%s_%s-.Lgpx_pf%s_%s" % (n, tag, n, tag), "s_addc_u32 s75, s75, 0",
         "s_sub_u32 s74, s74, s73", "s_subb_u32 s75, s75, 0", "s_setpc_b64 s[74:75]"]
    for k in range(PF_LINES, 0, -1):
        L += ["s_load_dword s79, s[58:59], 0x%x" % (64 * k)]
    return L + [".Lgpx_pfe%s_%s:" % (n, tag)]


def program_end(T, D, NF, V0, FO, tag, mode, ring):
    """End of a program: s66 holds its payload (low 24 bits: records of the
    program after it), s67 its row.  The next program's first records and
    lines are requested, the fitness terms of the tile are formed and summed
    over the wave in the fixed order, and the interpreter goes on."""
    m = V0 + T                       # stack levels above the result are free
    vl, vy, vo = m, m + 1, m + 1
    acc = [m + 2, m + 4]
    tmp = m + 6
    yr = m + 8
    assert yr + T <= V0 + FO
    y = lambda j: "v%d" % (yr + j)   # noqa: E731
    o = lambda j: "v%d" % (V0 + j)   # noqa: E731
    nb = T // 4
    full = 64 * T
    L = ["s_mov_b32 s80, s67", "s_and_b32 s81, s66, 0xffffff"] + ([] if ring else ["s_add_u32 s62, s62, 16"])
    L += ["v_mbcnt_lo_u32_b32 v%d, -1, 0" % vl, "v_mbcnt_hi_u32_b32 v%d, -1, v%d" % (vl, vl),
         "v_lshl_add_u32 v%d, v%d, 4, s97" % (vy, vl)]
    for k in range(nb):
        L += ["ds_read_b128 %s, v%d offset:%d" % (quad(yr + 4 * k), vy, 1024 * k)]
    L += ["s_waitcnt lgkmcnt(0)", first_records(ring, mode)[0],
          "s_lshl_b32 s81, s81, 4", "s_add_u32 s81, s81, s62"]
    L += prefetch_start(tag, "1", "s81")
    rows = ring and mode == 4
    if rows:
        L += ["s_cmp_eq_u32 s93, %d" % TO_ROW, "s_cbranch_scc1 .Lgpx_row_%s" % tag]
    kinds = [FIT_HITS, OUT_CASES] if mode == 2 else [FIT_MSE, FIT_SUM_ABS, FIT_HITS, FIT_CLASS, OUT_CASES]
    lab = {FIT_MSE: "mse", FIT_SUM_ABS: "abs", FIT_HITS: "hits", FIT_CLASS: "cls", OUT_CASES: "cases"}
    for k in kinds[1:]:
        L += ["s_cmp_eq_u32 s93, %d" % k, "s_cbranch_scc1 .Lgpx_%s_%s" % (lab[k], tag)]

    to_partials = ["s_mul_i32 s72, s80, s92", "s_mul_hi_u32 s73, s80, s92",
                   "s_add_u32 s80, s72, s90", "s_addc_u32 s81, s73, s91"]

    def store_sum():
        # one block: any lane holds the sum; two: lane 0 the first block's, lane 32 the second's
        if nb == 1:
            return ["v_mov_b32_e32 v%d, 0" % vo, "s_mov_b64 exec, 1",
                    "global_store_dwordx2 v%d, %s, s[80:81]" % (vo, pair(acc[0])), "s_mov_b64 exec, -1"]
        return ["v_lshrrev_b32_e32 v%d, 5, v%d" % (vo, vl), "v_lshlrev_b32_e32 v%d, 3, v%d" % (vo, vo),
                "s_cmp_gt_i32 s87, 256", "s_cselect_b32 s75, 1, 0", "s_mov_b32 s74, 1", "s_mov_b64 exec, s[74:75]",
                "global_store_dwordx2 v%d, %s, s[80:81]" % (vo, pair(acc[0])), "s_mov_b64 exec, -1"]

    def wave_sum():
        """The butterfly sum over lanes 32, 16, 8, 4, 2, 1 apart, without LDS:
        half and row exchanges (v_permlane*_swap), then rotations within a row
        and a quad, which reach the same partner once the wider steps have
        made the values equal."""
        S = []
        a, t = acc[0], tmp
        if nb == 1:
            S += ["v_mov_b32_e32 v%d, v%d" % (t, a), "v_mov_b32_e32 v%d, v%d" % (t + 1, a + 1)]
        else:
            t = acc[1]
        S += ["s_nop 1", "v_permlane32_swap_b32 v%d, v%d" % (a, t), "v_permlane32_swap_b32 v%d, v%d" % (a + 1, t + 1),
              "s_nop 1", "v_add_f64 %s, %s, %s" % (pair(a), pair(a), pair(t))]
        t = tmp
        S += ["v_mov_b32_e32 v%d, v%d" % (t, a), "v_mov_b32_e32 v%d, v%d" % (t + 1, a + 1), "s_nop 1",
              "v_permlane16_swap_b32 v%d, v%d" % (a, t), "v_permlane16_swap_b32 v%d, v%d" % (a + 1, t + 1),
              "s_nop 1", "v_add_f64 %s, %s, %s" % (pair(a), pair(a), pair(t))]
        for ctl in ("row_ror:8", "row_ror:4", "quad_perm:[2,3,0,1]", "quad_perm:[1,0,3,2]"):
            S += ["s_nop 1", "v_mov_b32_dpp v%d, v%d %s row_mask:0xf bank_mask:0xf" % (t, a, ctl),
                  "v_mov_b32_dpp v%d, v%d %s row_mask:0xf bank_mask:0xf" % (t + 1, a + 1, ctl),
                  "v_add_f64 %s, %s, %s" % (pair(a), pair(a), pair(t))]
        return S

    done = ["s_branch .Lgpx_next_%s" % tag]
    for k in kinds:
        name = lab[k]
        if k != kinds[0]:
            L += [".Lgpx_%s_%s:" % (name, tag)]
        if k == OUT_CASES:
            L += ["v_lshlrev_b32_e32 v%d, 2, v%d" % (vl, vl),
                  "s_mul_i32 s72, s80, s84", "s_mul_hi_u32 s73, s80, s84", "s_mul_i32 s74, s80, s85",
                  "s_add_u32 s73, s73, s74", "s_add_u32 s80, s72, s94", "s_addc_u32 s81, s73, s95"]
            for j in range(T):
                L += exec_slot(j)
                L += ["global_store_dword v%d, %s, s[80:81] offset:%d" % (vl, o(j), 256 * j)]
            L += ["s_mov_b64 exec, -1"] + done
            continue
        L += to_partials
        if k in (FIT_MSE, FIT_SUM_ABS):
            cvt = (lambda d, s: "v_cvt_f64_f32_e32 %s, %s" % (pair(d), s)) if k == FIT_MSE else \
                (lambda d, s: "v_cvt_f64_f32_e64 %s, |%s|" % (pair(d), s))
            for j in range(T):
                L += ["v_sub_f32_e32 %s, %s, %s" % (o(j), o(j), y(j))]
                if k == FIT_MSE:
                    L += ["v_mul_f32_e32 %s, %s, %s" % (o(j), o(j), o(j))]
            L += ["s_cmp_lt_i32 s87, %d" % full, "s_cbranch_scc1 .Lgpx_r%s_%s" % (name, tag)]
            for b in range(nb):
                L += [cvt(acc[b], o(4 * b))]
                for j in range(4 * b + 1, 4 * b + 4):
                    L += [cvt(tmp, o(j)), "v_add_f64 %s, %s, %s" % (pair(acc[b]), pair(acc[b]), pair(tmp))]
            L += [".Lgpx_w%s_%s:" % (name, tag)] + wave_sum()
        elif mode == 2:
            # words: matching bits, counted per lane, then over the row and the wave (whole numbers: any order)
            L += ["s_cmp_lt_u32 s98, %d" % (32 * full), "s_cbranch_scc1 .Lgpx_r%s_%s" % (name, tag)]
            for j in range(T):
                L += ["v_xnor_b32_e32 %s, %s, %s" % (o(j), o(j), y(j))]
            L += [".Lgpx_w%s_%s:" % (name, tag)]
            for b in range(nb):
                L += ["v_bcnt_u32_b32 v%d, %s, 0" % (acc[b], o(4 * b))]
                for j in range(4 * b + 1, 4 * b + 4):
                    L += ["v_bcnt_u32_b32 v%d, %s, v%d" % (acc[b], o(j), acc[b])]
            for b in range(nb):
                for ctl in ("row_ror:8", "row_ror:4", "row_ror:2", "row_ror:1"):
                    L += ["s_nop 1", "v_add_u32_dpp v%d, v%d, v%d %s row_mask:0xf bank_mask:0xf"
                          % (acc[b], acc[b], acc[b], ctl)]
            L += ["s_nop 1"]
            for b in range(nb):
                L += ["v_readlane_b32 s72, v%d, 0" % acc[b], "v_readlane_b32 s73, v%d, 16" % acc[b],
                      "v_readlane_b32 s74, v%d, 32" % acc[b], "v_readlane_b32 s75, v%d, 48" % acc[b],
                      "s_add_u32 s72, s72, s73", "s_add_u32 s74, s74, s75", "s_add_u32 s%d, s72, s74" % (77 if b else 76)]
            L += count_out(nb, acc, tmp)
        else:
            L += ["s_cmp_lt_i32 s87, %d" % full, "s_cbranch_scc1 .Lgpx_r%s_%s" % (name, tag)]
            L += hit_terms(k, T, o, y, False)
            L += [".Lgpx_w%s_%s:" % (name, tag)] + count_out(nb, acc, tmp)
        L += store_sum() + done
    # ragged tiles (and, for Boolean programs, the data's last words)
    for k in kinds:
        name = lab[k]
        if k == OUT_CASES:
            continue
        L += [".Lgpx_r%s_%s:" % (name, tag)]
        if k in (FIT_MSE, FIT_SUM_ABS):
            for b in range(nb):
                L += ["v_mov_b32_e32 v%d, 0" % acc[b], "v_mov_b32_e32 v%d, 0" % (acc[b] + 1)]
            for j in range(T):
                a = acc[j // 4]
                cv = "v_cvt_f64_f32_e32 %s, %s" % (pair(tmp), o(j)) if k == FIT_MSE else \
                    "v_cvt_f64_f32_e64 %s, |%s|" % (pair(tmp), o(j))
                L += exec_slot(j) + [cv, "v_add_f64 %s, %s, %s" % (pair(a), pair(a), pair(tmp))]
            L += ["s_mov_b64 exec, -1"]
        elif mode == 2:
            # bits left in the word of slot j: s98 - 32 (64 j + lane), as a mask of 0 .. 32 low bits
            L += ["v_lshlrev_b32_e32 v%d, 5, v%d" % (tmp, vl), "v_sub_u32_e32 v%d, s98, v%d" % (tmp, tmp)]
            for j in range(T):
                L += ["v_add_u32_e32 v%d, 0x%x, v%d" % (tmp + 1, (-2048 * j) & 0xFFFFFFFF, tmp),
                      "v_med3_i32 v%d, v%d, 0, 32" % (tmp + 1, tmp + 1),
                      "v_sub_u32_e32 v%d, 32, v%d" % (tmp + 1, tmp + 1),
                      # ~0 >> (32 - bits); the shift takes 5 bits, so no bits at all is patched to 0
                      "v_lshrrev_b32_e64 v%d, v%d, -1" % (vo, tmp + 1),
                      "v_cmp_gt_u32_e32 vcc, 32, v%d" % (tmp + 1),
                      "v_xnor_b32_e32 %s, %s, %s" % (o(j), o(j), y(j)), "s_nop 1",
                      "v_cndmask_b32_e32 v%d, 0, v%d, vcc" % (vo, vo),
                      "v_and_b32_e32 %s, %s, v%d" % (o(j), o(j), vo)]
        else:
            L += hit_terms(k, T, o, y, True)
            L += ["s_mov_b64 exec, -1"]
        L += ["s_branch .Lgpx_w%s_%s" % (name, tag)]
    if rows:
        L += [".Lgpx_row_%s:" % tag, "s_lshl_b32 s72, s80, %d" % (8 + T.bit_length() - 1),
              "v_lshl_add_u32 v%d, v%d, 4, s72" % (vy, vl),
              "ds_write_b128 v%d, %s offset:%d" % (vy, quad(V0), rows_base(T, D, NF, V0, mode))]
        assert T == 4
    L += [".Lgpx_next_%s:" % tag, "s_cmp_ge_u32 s62, s96", "s_cbranch_scc0 .Lgpx_rest_%s" % tag]
    if rows:
        L += ["s_cmp_eq_u32 s98, -1", "s_cbranch_scc1 .Lgpx_probe_%s" % tag, "s_waitcnt lgkmcnt(0)", "s_barrier",
              "s_mov_b32 s62, s56", "s_mov_b32 s96, s57", "s_mov_b32 s93, s98", "s_mov_b32 s98, -1",
              "s_cmp_ge_u32 s62, s96", "s_cbranch_scc1 .Lgpx_probe_%s" % tag, first_records(ring, mode)[0]]
        L += prefetch_start(tag, "3", "s96") + ["s_mov_b32 s99, 0", "s_branch .Lgpx_rest_%s" % tag]
    L += [".Lgpx_probe_%s:" % tag, "s_branch .Lgpx_leave_%s" % tag]
    L += [".Lgpx_rest_%s:" % tag, "s_waitcnt lgkmcnt(0)", "s_cmp_eq_u32 s99, 0", "s_cbranch_scc1 .Lgpx_go_%s" % tag,
          "s_lshl_b32 s72, s78, 6", "s_add_u32 s58, s58, s72", "s_addc_u32 s59, s59, 0"]
    L += prefetch_lines(tag, "2")
    L += ["s_branch .Lgpx_rest_%s" % tag, ".Lgpx_go_%s:" % tag] + first_records(ring, mode)[1]
    return L


def hit_terms(kind, T, o, y, ragged):
    """Counts of a block's hits (sign rule) or class errors (rint(o) is not the class), into s[76 + block]."""
    L = []
    for j in range(T):
        cnt = "s%d" % (76 + j // 4)
        if ragged:
            # a compare writes 0 for the lanes outside exec
            L += exec_slot(j)
        if kind == FIT_HITS:
            L += ["v_cmp_lt_f32_e32 vcc, 0, %s" % o(j), "v_cmp_lt_f32_e64 s[72:73], 0, %s" % y(j),
                  "s_xnor_b64 s[72:73], vcc, s[72:73]"]
            if ragged:
                L += ["s_and_b64 s[72:73], s[72:73], exec"]
        else:
            L += ["v_rndne_f32_e32 %s, %s" % (o(j), o(j)), "v_cmp_neq_f32_e64 s[72:73], %s, %s" % (o(j), y(j))]
        if j % 4 == 0:
            L += ["s_bcnt1_i32_b64 %s, s[72:73]" % cnt]
        else:
            L += ["s_bcnt1_i32_b64 s74, s[72:73]", "s_add_u32 %s, %s, s74" % (cnt, cnt)]
    return L


def count_out(nb, acc, tmp):
    """Block counts in s76 (and s77) as binary64, where store_sum takes them."""
    L = ["v_mov_b32_e32 v%d, s76" % tmp]
    if nb == 2:
        L += ["s_mov_b32 s74, 0", "s_mov_b32 s75, -1", "s_mov_b64 exec, s[74:75]", "v_mov_b32_e32 v%d, s77" % tmp,
              "s_mov_b64 exec, -1"]
    return L + ["v_cvt_f64_u32_e32 %s, v%d" % (pair(acc[0]), tmp)]


def transc(T, V0, NCV, tag, mode, ring):
    """sin, cos, exp and log of T slots (s72 the operation, s66 the payload,
    s67 a constant operand): the arithmetic of gp_math.h, instruction by
    instruction, in the block's work registers, with operand and result
    through the index mode and no copies for cos and log.  The record pair
    after the exit is loaded meanwhile."""
    n = transc_slots(NCV)
    w0 = V0 - 14 * n - 2
    G = V0 - 2                                  # a pair shared by the slots (large arguments)
    keep = NCV >= 64

    def reg(i):
        b = w0 + 14 * i                          # X r V C D(4) E a
        return dict(X=b, R=b + 2, V=b + 4, C=b + 6, D=b + 8, E=b + 12, a=b + 13)

    names = list(VCONST)

    def vc(nm):                                  # register of a VGPR constant
        return vconst_reg(V0, mode, names.index(nm)) if keep else None

    def coef(nm):
        return sp(COEF[nm])
    L = [".Lgpx_fn_%s:" % tag, "s_and_b32 s73, s66, 0xff", "s_bfe_u32 s79, s66, 0x80010", "s_bitcmp1_b32 s66, 28",
         "s_cbranch_scc0 .Lgpx_fa_%s" % tag, "s_set_gpr_idx_on s79, gpr_idx(DST)"]
    L += ["v_mov_b32_e32 v%d, s67" % (V0 + j) for j in range(T)]
    L += ["s_set_gpr_idx_off", "s_mov_b32 s73, s79", ".Lgpx_fa_%s:" % tag]
    L += ["s_waitcnt lgkmcnt(0)"] if ring else ["s_add_u32 s62, s62, 16"]
    L += [first_records(ring, mode)[0],
          "s_cmp_eq_u32 s72, 6", "s_cbranch_scc1 .Lgpx_exp_%s" % tag,
          "s_cmp_eq_u32 s72, 7", "s_cbranch_scc1 .Lgpx_log_%s" % tag,
          "s_cmp_eq_u32 s72, 5", "s_cbranch_scc1 .Lgpx_cos_%s" % tag]
    fin = ["s_waitcnt lgkmcnt(0)"] + first_records(ring, mode)[1]
    out_of_line = []

    def const(nm, into):
        """A VGPR constant's register: kept, or moved into `into` now."""
        if keep:
            return pair(vc(nm)), []
        hi, lo = VCONST[nm]
        return pair(into), ["v_mov_b32_e32 v%d, 0x%x" % (into, lo), "v_mov_b32_e32 v%d, 0x%x" % (into + 1, hi)]

    def weave(seqs):
        out = []
        for k in range(max(len(x) for x in seqs)):
            out += [x[k] for x in seqs if k < len(x)]
        return out

    def idx(sreg, field, body):
        return ["s_set_gpr_idx_on %s, gpr_idx(%s)" % (sreg, field)] + body + ["s_set_gpr_idx_off"]

    for fn in ("sin", "cos"):
        if fn == "cos":
            L += [".Lgpx_cos_%s:" % tag]
        for g in range(0, T, n):
            rs = [reg(i) for i in range(n)]
            src = ["v%d" % (V0 + g + i) for i in range(n)]
            if fn == "sin":
                L += idx("s73", "SRC0", ["v_mov_b32_e32 v%d, %s" % (r["a"], s) for r, s in zip(rs, src)])
                L += ["v_cvt_f64_f32_e32 %s, v%d" % (pair(r["X"]), r["a"]) for r in rs]
            else:
                L += idx("s73", "SRC0", ["v_cvt_f64_f32_e32 %s, %s" % (pair(r["X"]), s) for r, s in zip(rs, src)])
            seqs = []
            for r in rs:
                q = []
                R, mv = const("R", r["C"])
                q += mv
                q += ["v_fma_f64 %s, %s, %s, %s" % (pair(r["V"]), pair(r["X"]), coef("KPI"), R),
                      "v_add_f64 %s, %s, -%s" % (pair(r["C"]), pair(r["V"]), R),
                      "v_fma_f64 %s, -%s, %s, %s" % (pair(r["R"]), pair(r["C"]), coef("P1"), pair(r["X"])),
                      "v_fma_f64 %s, -%s, %s, %s" % (pair(r["R"]), pair(r["C"]), coef("P2"), pair(r["R"])),
                      "v_fma_f64 %s, -%s, %s, %s" % (pair(r["R"]), pair(r["C"]), coef("P3"), pair(r["R"]))]
                seqs.append(q)
            L += weave(seqs)
            # any argument of 2^44 or more (its high word; the sign shifted out): another reduction
            big, back = ".Lgpx_big_%s%d_%s" % (fn, g, tag), ".Lgpx_red_%s%d_%s" % (fn, g, tag)
            if n == 2:
                L += ["v_max_f64 %s, |%s|, |%s|" % (pair(rs[0]["D"]), pair(rs[0]["X"]), pair(rs[1]["X"]))]
                L += ["v_cmp_lt_u32_e32 vcc, 0x42afffff, v%d" % (rs[0]["D"] + 1)]
            else:
                L += ["v_and_b32_e32 v%d, 0x7fffffff, v%d" % (rs[0]["D"], rs[0]["X"] + 1),
                      "v_cmp_lt_u32_e32 vcc, 0x42afffff, v%d" % rs[0]["D"]]
            L += ["s_cbranch_vccnz %s" % big, "%s:" % back]
            out_of_line += ["%s:" % big]
            for r in rs:
                out_of_line += big_reduction(r, G)
            out_of_line += ["s_branch %s" % back]
            seqs = []
            for r in rs:
                q = ["v_lshlrev_b32_e32 v%d, 4, v%d" % (r["V"], r["V"])]
                if fn == "cos":      # a quarter turn on: entry j + 32
                    q = ["v_lshlrev_b32_e32 v%d, 4, v%d" % (r["V"], r["V"]), "v_add_u32_e32 v%d, 0x200, v%d" % (r["V"], r["V"])]
                q += ["v_and_b32_e32 v%d, 0x7f0, v%d" % (r["V"], r["V"]),
                      "ds_read_b128 %s, v%d offset:%d" % (quad(r["D"]), r["V"], LDS_SC),
                      "v_mul_f64 %s, %s, %s" % (pair(r["C"]), pair(r["R"]), pair(r["R"]))]
                S1, mv = const("S1", r["V"])
                q += mv + ["v_fma_f64 %s, %s, %s, %s" % (pair(r["X"]), pair(r["C"]), coef("S2"), S1),
                           "v_fma_f64 %s, %s, %s, %s" % (pair(r["X"]), pair(r["X"]), pair(r["C"]), coef("S0"))]
                C1, mv = const("C1", r["V"])
                tv = pair(r["V"])
                q += mv + ["v_fma_f64 %s, %s, %s, %s" % (tv, pair(r["C"]), coef("C2"), C1),
                           "v_fma_f64 %s, %s, %s, -0.5" % (tv, tv, pair(r["C"])),
                           "v_fma_f64 %s, %s, %s, 1.0" % (tv, tv, pair(r["C"])),            # cos r
                           "v_mul_f64 %s, %s, %s" % (pair(r["C"]), pair(r["R"]), pair(r["C"])),
                           "v_fma_f64 %s, %s, %s, %s" % (pair(r["R"]), pair(r["C"]), pair(r["X"]), pair(r["R"]))]  # sin r
                seqs.append(q)
            L += weave(seqs) + ["s_waitcnt lgkmcnt(0)"]
            seqs = []
            for r in rs:
                seqs.append(["v_mul_f64 %s, %s, %s" % (pair(r["R"]), pair(r["D"] + 2), pair(r["R"])),
                             "v_fma_f64 %s, %s, %s, %s" % (pair(r["R"]), pair(r["D"]), pair(r["V"]), pair(r["R"]))])
            L += weave(seqs)
            if fn == "sin":
                for r in rs:
                    L += ["v_cvt_f32_f64_e32 v%d, %s" % (r["V"], pair(r["R"]))]
                L += ["s_mov_b32 s80, 0x39800000"]            # |a| below 2^-12: a itself
                for i, r in enumerate(rs):
                    L += ["v_cmp_lt_f32_e64 s[%d:%d], |v%d|, s80" % (74 + 2 * i, 75 + 2 * i, r["a"])]
                L += ["s_nop 1"]
                L += idx("s79", "DST", ["v_cndmask_b32_e64 %s, v%d, v%d, s[%d:%d]" % (s, r["V"], r["a"], 74 + 2 * i, 75 + 2 * i)
                                        for i, (r, s) in enumerate(zip(rs, src))])
            else:
                L += idx("s79", "DST", ["v_cvt_f32_f64_e32 %s, %s" % (s, pair(r["R"])) for r, s in zip(rs, src)])
        L += fin
    L += [".Lgpx_exp_%s:" % tag, "s_mov_b32 s80, 0xc2d00000", "s_mov_b32 s81, 0x42b00000"]
    for g in range(0, T, n):
        rs = [reg(i) for i in range(n)]
        src = ["v%d" % (V0 + g + i) for i in range(n)]
        L += idx("s73", "SRC0", ["v_mov_b32_e32 v%d, %s" % (r["a"], s) for r, s in zip(rs, src)])
        seqs = []
        for r in rs:
            # clamped to [-104, 88]; a NaN is put back at the end
            q = ["v_max_f32_e32 v%d, s80, v%d" % (r["E"], r["a"]), "v_min_f32_e32 v%d, s81, v%d" % (r["E"], r["E"]),
                 "v_cvt_f64_f32_e32 %s, v%d" % (pair(r["X"]), r["E"])]
            R, mv = const("R", r["C"])
            q += mv + ["v_fma_f64 %s, %s, %s, %s" % (pair(r["V"]), pair(r["X"]), coef("KLN"), R),
                       "v_add_f64 %s, %s, -%s" % (pair(r["C"]), pair(r["V"]), R),
                       "v_lshlrev_b32_e32 v%d, 3, v%d" % (r["E"], r["V"]), "v_and_b32_e32 v%d, 0x1f8, v%d" % (r["E"], r["E"]),
                       "ds_read_b64 %s, v%d offset:%d" % (pair(r["D"]), r["E"], LDS_EXP),
                       "v_fma_f64 %s, -%s, %s, %s" % (pair(r["X"]), pair(r["C"]), coef("L1"), pair(r["X"])),
                       "v_fma_f64 %s, -%s, %s, %s" % (pair(r["X"]), pair(r["C"]), coef("L2"), pair(r["X"])),
                       "v_ashrrev_i32_e32 v%d, 6, v%d" % (r["E"], r["V"])]
            E2, mv = const("E2", r["C"])
            t = pair(r["R"])
            q += mv + ["v_fma_f64 %s, %s, %s, %s" % (t, pair(r["X"]), coef("E3"), E2),
                       "v_fma_f64 %s, %s, %s, %s" % (t, t, pair(r["X"]), coef("E1")),
                       "v_fma_f64 %s, %s, %s, 0.5" % (t, t, pair(r["X"])),
                       "v_fma_f64 %s, %s, %s, 1.0" % (t, t, pair(r["X"])),
                       "v_fma_f64 %s, %s, %s, 1.0" % (t, t, pair(r["X"]))]
            seqs.append(q)
        L += weave(seqs) + ["s_waitcnt lgkmcnt(0)"]
        seqs = [["v_mul_f64 %s, %s, %s" % (pair(r["R"]), pair(r["D"]), pair(r["R"])),
                 "v_ldexp_f64 %s, %s, v%d" % (pair(r["R"]), pair(r["R"]), r["E"]),
                 "v_cvt_f32_f64_e32 v%d, %s" % (r["V"], pair(r["R"])),
                 "v_cmp_u_f32_e64 s[%d:%d], v%d, v%d" % (74 + 2 * i, 75 + 2 * i, r["a"], r["a"])] for i, r in enumerate(rs)]
        L += weave(seqs) + ["s_nop 1"]
        L += idx("s79", "DST", ["v_cndmask_b32_e64 %s, v%d, v%d, s[%d:%d]" % (s, r["V"], r["a"], 74 + 2 * i, 75 + 2 * i)
                                for i, (r, s) in enumerate(zip(rs, src))])
    L += fin
    L += [".Lgpx_log_%s:" % tag, "s_mov_b32 s80, 0x%x" % DIV_THRESHOLD, "s_mov_b32 s81, 0x7f800000"]
    c0 = (0x3F3504F3 + 0x4000 - (LOG_K0 << 15)) & 0xFFFFFFFF
    for g in range(0, T, n):
        rs = [reg(i) for i in range(n)]
        src = ["v%d" % (V0 + g + i) for i in range(n)]
        L += idx("s73", "SRC1", ["v_and_b32_e32 v%d, 0x7fffffff, %s" % (r["a"], s) for r, s in zip(rs, src)])
        seqs = []
        for r in rs:
            # the encoding relative to sqrt(1/2): exponent e, f in [sqrt(1/2), sqrt(2)), its bucket's table entry;
            # any encoding gives a valid bucket, so zeros, infinities and NaN are put right at the end
            q = ["v_add_u32_e32 v%d, 0x%x, v%d" % (r["V"], (-0x3F3504F3) & 0xFFFFFFFF, r["a"]),
                 "v_ashrrev_i32_e32 v%d, 23, v%d" % (r["E"], r["V"]),
                 "v_and_b32_e32 v%d, 0x7fffff, v%d" % (r["V"], r["V"]),
                 "v_add_u32_e32 v%d, 0x%x, v%d" % (r["V"] + 1, c0, r["V"]),
                 "v_lshrrev_b32_e32 v%d, 11, v%d" % (r["V"] + 1, r["V"] + 1),
                 "v_and_b32_e32 v%d, 0xfffffff0, v%d" % (r["V"] + 1, r["V"] + 1),
                 "ds_read_b128 %s, v%d offset:%d" % (quad(r["D"]), r["V"] + 1, LDS_LOG),
                 "v_add_u32_e32 v%d, 0x3f3504f3, v%d" % (r["V"], r["V"]),
                 "v_cvt_f64_f32_e32 %s, v%d" % (pair(r["X"]), r["V"]),
                 "v_cvt_f64_i32_e32 %s, v%d" % (pair(r["R"]), r["E"])]
            seqs.append(q)
        L += weave(seqs) + ["s_waitcnt lgkmcnt(0)"]
        seqs = []
        for i, r in enumerate(rs):
            G3, mv = const("G3", r["C"])
            t = pair(r["V"])
            q = ["v_fma_f64 %s, %s, %s, -1.0" % (pair(r["X"]), pair(r["X"]), pair(r["D"]))]
            q += mv + ["v_fma_f64 %s, %s, %s, %s" % (t, pair(r["X"]), coef("G4"), G3),
                       "v_fma_f64 %s, %s, %s, %s" % (t, t, pair(r["X"]), coef("G2")),
                       "v_fma_f64 %s, %s, %s, %s" % (t, t, pair(r["X"]), coef("G1")),
                       "v_fma_f64 %s, %s, %s, -0.5" % (t, t, pair(r["X"])),
                       "v_mul_f64 %s, %s, %s" % (pair(r["C"]), pair(r["X"]), pair(r["X"])),
                       "v_fma_f64 %s, %s, %s, %s" % (t, pair(r["C"]), t, pair(r["X"])),
                       "v_add_f64 %s, %s, %s" % (t, pair(r["D"] + 2), t),
                       "v_fma_f64 %s, %s, %s, %s" % (t, pair(r["R"]), coef("LN2"), t),
                       "v_cvt_f32_f64_e32 v%d, %s" % (r["V"], t),
                       "v_cmp_gt_u32_e64 s[%d:%d], s81, v%d" % (74 + 2 * i, 75 + 2 * i, r["a"]), "s_nop 1",
                       "v_cndmask_b32_e64 v%d, v%d, v%d, s[%d:%d]" % (r["V"], r["a"], r["V"], 74 + 2 * i, 75 + 2 * i),
                       "v_cmp_gt_f32_e64 s[%d:%d], s80, v%d" % (74 + 2 * i, 75 + 2 * i, r["a"])]
            seqs.append(q)
        L += weave(seqs) + ["s_nop 1"]
        L += idx("s79", "DST", ["v_cndmask_b32_e64 %s, v%d, 0, s[%d:%d]" % (s, r["V"], 74 + 2 * i, 75 + 2 * i)
                                for i, (r, s) in enumerate(zip(rs, src))])
    L += fin
    return L + out_of_line


def big_reduction(r, G):
    """x mod 2 pi for the lanes with |x| >= 2^44 (gp_math.h, reduce_big):
    r and the low word of V (k) are replaced there.  E: 37 n >> 10 is n div 28
    for n up to 103."""
    X, A, P2, K = pair(r["X"]), pair(r["C"]), pair(r["D"] + 2), pair(G)
    D = pair(r["D"])
    E = "v%d" % r["E"]
    v1 = pair(r["D"])
    L = ["v_cvt_f32_f64_e64 %s, |%s|" % (E, X),
         "v_lshrrev_b32_e32 %s, 23, %s" % (E, E), "v_max_u32_e32 %s, 0xab, %s" % (E, E),
         "v_subrev_u32_e32 %s, 0x98, %s" % (E, E), "v_mul_u32_u24_e32 %s, 37, %s" % (E, E),
         "v_lshrrev_b32_e32 %s, 10, %s" % (E, E), "v_lshlrev_b32_e32 %s, 3, %s" % (E, E),
         # v0 in C
         "ds_read_b64 %s, %s offset:%d" % (A, E, LDS_PI), "s_waitcnt lgkmcnt(0)",
         "v_mul_f64 %s, |%s|, %s" % (A, X, A), "v_ldexp_f64 %s, %s, -7" % (K, A), "v_floor_f64_e32 %s, %s" % (K, K),
         "v_ldexp_f64 %s, -%s, 7" % (K, K), "v_add_f64 %s, %s, %s" % (A, K, A),
         # v1 in D
         "ds_read_b64 %s, %s offset:%d" % (v1, E, LDS_PI + 8), "s_waitcnt lgkmcnt(0)",
         "v_mul_f64 %s, |%s|, %s" % (v1, X, v1), "v_ldexp_f64 %s, %s, -7" % (K, v1), "v_floor_f64_e32 %s, %s" % (K, K),
         "v_ldexp_f64 %s, -%s, 7" % (K, K), "v_add_f64 %s, %s, %s" % (v1, K, v1),
         # p2, and kd = rint(v0 + v1 + p2)
         "ds_read_b64 %s, %s offset:%d" % (P2, E, LDS_PI + 16), "s_waitcnt lgkmcnt(0)",
         "v_mul_f64 %s, |%s|, %s" % (P2, X, P2),
         "v_add_f64 %s, %s, %s" % (K, A, v1), "v_add_f64 %s, %s, %s" % (K, K, P2), "v_rndne_f64_e32 %s, %s" % (K, K),
         # s = (((v0 - kd) + v1) + p2 + p3) + p4
         "v_add_f64 %s, %s, -%s" % (A, A, K), "v_add_f64 %s, %s, %s" % (A, A, v1), "v_add_f64 %s, %s, %s" % (A, A, P2),
         "ds_read_b64 %s, %s offset:%d" % (v1, E, LDS_PI + 24), "ds_read_b64 %s, %s offset:%d" % (P2, E, LDS_PI + 32),
         "s_waitcnt lgkmcnt(0)",
         "v_mul_f64 %s, |%s|, %s" % (v1, X, v1), "v_mul_f64 %s, |%s|, %s" % (P2, X, P2),
         "v_add_f64 %s, %s, %s" % (A, A, v1), "v_add_f64 %s, %s, %s" % (A, A, P2),
         "v_mul_f64 %s, %s, %s" % (A, A, sp(COEF["P1"])),
         # the sign of x, on r and k
         "v_and_b32_e32 %s, 0x80000000, v%d" % (E, r["X"] + 1),
         "v_xor_b32_e32 v%d, %s, v%d" % (r["C"] + 1, E, r["C"] + 1), "v_xor_b32_e32 v%d, %s, v%d" % (G + 1, E, G + 1),
         "v_cvt_i32_f64_e32 v%d, %s" % (G, K),
         "v_and_b32_e32 %s, 0x7fffffff, v%d" % (E, r["X"] + 1), "v_cmp_lt_u32_e32 vcc, 0x42afffff, %s" % E, "s_nop 1",
         "v_cndmask_b32_e32 v%d, v%d, v%d, vcc" % (r["R"], r["R"], r["C"]),
         "v_cndmask_b32_e32 v%d, v%d, v%d, vcc" % (r["R"] + 1, r["R"] + 1, r["C"] + 1),
         "v_cndmask_b32_e32 v%d, v%d, v%d, vcc" % (r["V"], r["V"], G)]
    return L


def load_feature(T, V0, tag, mode):
    """A feature of the tile (its number in s66) into stack level 0, for the programs of the rows."""
    vl = "v%d" % (V0 + T)                        # stack level 1 is free here
    L = [".Lgpx_ldf_%s:" % tag, "s_waitcnt lgkmcnt(0)", first_records(True, mode)[0],
         "s_and_b32 s80, s66, 0xffffff",
         "s_mul_i32 s76, s80, s84", "s_mul_hi_u32 s77, s80, s84", "s_mul_i32 s81, s80, s85", "s_add_u32 s77, s77, s81",
         "s_add_u32 s76, s76, s82", "s_addc_u32 s77, s77, s83",
         "v_mbcnt_lo_u32_b32 %s, -1, 0" % vl, "v_mbcnt_hi_u32_b32 %s, -1, %s" % (vl, vl), "v_lshlrev_b32_e32 %s, 2, %s" % (vl, vl)]
    for j in range(T):
        L += exec_slot(j) + ["global_load_dword v%d, %s, s[76:77] offset:%d" % (V0 + j, vl, 256 * j)]
    return L + ["s_mov_b64 exec, -1", "s_waitcnt vmcnt(0) lgkmcnt(0)"] + first_records(True, mode)[1]


def tail_lines(T, D, NF, V0, FO, tag, mode, ring):
    """What follows the handlers in the block: an exit's record is in s[66:67]."""
    L = [".Lgpx_end_%s:" % tag]
    if mode in (0, 4):
        L += ["s_bfe_u32 s72, s66, 0x40018"]
        if (T, D, NF, V0, mode) in WIDE and ring:
            L += ["s_cmp_eq_u32 s72, 14", "s_cbranch_scc1 .Lgpx_ldf_%s" % tag]
        L += ["s_cmp_lg_u32 s72, 15", "s_cbranch_scc1 .Lgpx_fn_%s" % tag]
    L += program_end(T, D, NF, V0, FO, tag, mode, ring)
    if mode in (0, 4):
        L += transc(T, V0, V0, tag, mode, ring)
    if (T, D, NF, V0, mode) in WIDE and ring:
        L += load_feature(T, V0, tag, mode)
    if ring and mode != 2:
        L += division_bodies(T, D, V0, tag)
    L += [".Lgpx_leave_%s:" % tag, "s_waitcnt vmcnt(0) lgkmcnt(0)"]
    return L


def asm_text(T, D, NF, V0, FO, tag, hs, mode, ring=False):
    slot = RING_SLOT if ring else SLOT
    L = []
    L.append("s_getpc_b64 s[76:77]")
    L.append(".Lgpx_pc_%s:" % tag)
    L.append("s_cmp_eq_u32 s63, 0")
    L.append("s_cbranch_scc1 .Lgpx_run_%s" % tag)
    L.append("s_add_u32 s76, s76, .Lgpx_table_%s-.Lgpx_pc_%s" % (tag, tag))
    L.append("s_addc_u32 s77, s77, 0")
    L.append("s_branch .Lgpx_probe_%s" % tag)
    L.append(".Lgpx_run_%s:" % tag)
    L += unit_start(T, D, NF, V0, FO, tag, mode, ring)
    L.append(".p2align %d" % (SLOT.bit_length() - 1))
    L.append(".Lgpx_table_%s:" % tag)
    for i, h in enumerate(hs):
        lab = ".Lgpx_h%d_%s" % (i, tag)
        L.append("%s:" % lab)
        # the host addresses handlers by slot: check the slot arithmetic
        L.append(".if (%s - .Lgpx_table_%s) != %d" % (lab, tag, h.slot * slot))
        L.append('.error \\"gpx handler %d misplaced\\"' % i)
        L.append(".endif")
        L.extend(h.lines)
        # pad to the slot boundary (never executed: every handler ends in a jump)
        pad = (-h.size) % slot
        L.extend(["s_nop 0"] * (pad // 4))
    L += tail_lines(T, D, NF, V0, FO, tag, mode, ring)
    # one string literal a line: the compiler locates each line of one long literal anew from its start
    return "\\n\\t\"\n            \"".join(L)


def relabelled(hs, tag):
    """The handlers with their jumps to this block's own labels (two kernels may share a handler table's layout)."""
    import re
    out = []
    for h in hs:
        c = Handler(h.kind, h.op, h.p1, h.p2)
        c.lines, c.size, c.slot = [re.sub(r"(\.Lgpx_[a-z]+\d*_)\w+", r"\g<1>" + tag, x) for x in h.lines], h.size, h.slot
        out.append(c)
    return out


def main(out_dir):
    os.makedirs(out_dir, exist_ok=True)
    lines = ["// Generated by gen_core.py -- do not edit.", "#pragma once", ""]
    lines.append("#define GPX_LIN_REGS %d" % LIN_REGS)
    lines.append("#define GPX_SLOT %d" % SLOT)
    lines.append("#define GPX_RING_PHASE %d" % RING_PHASE)
    lines.append("enum CoreKind {" + ", ".join("CK_%s = %d" % (k, i) for i, k in enumerate(KINDS)) + "};")
    lines.append("")
    lines.append("#define GPX_CORE_VARIANTS(X) \\")
    lines.append(" \\\n".join("    X(%d, %d, %d, %d, %d)" % v for v in VARIANTS))
    lines.append("")
    cores = []
    lines.append("template <int T, int D, int NF, int V0, int K> struct Core;   // K: kernel mode")
    lines.append("struct CoreUnit {")
    lines.append("    uint64_t code, X, stride, y, partials, cases, coef;")
    lines.append("    uint32_t off, end, n_load, left, part_stride, kind, lds_y, bits, burst;")
    lines.append("    uint32_t own_off, own_end, own_kind;   // after the rows (ring cores with sin/cos/exp/log)")
    lines.append("};")
    host = []
    seen = {}
    for vi, (T, D, NF, NCV, AR) in enumerate(VARIANTS + RING_VARIANTS):
        core = (T, D, NF, NCV, AR)
        ring = vi >= len(VARIANTS)
        assert core not in (VARIANTS + RING_VARIANTS)[:vi], core
        tag, V0, FO, hs, nslots = gen_variant(T, D, NF, NCV, AR, ring)
        tag += ("A" if AR == 1 else "S" if AR == 4 else "") + ("Q" if ring else "")
        key = (T, D, NF, NCV, {1: 0, 4: 3}.get(AR, AR), ring)    # modes 0 and 1 share a handler table, so do 3 and 4
        hs_tag, hs, nslots = seen.setdefault(key, (tag, hs, nslots))
        text = asm_text(T, D, NF, V0, FO, tag, relabelled(hs, tag), AR, ring)
        assert NCV + FO + NF * T <= 256
        work = work_regs(NCV, AR, ring)
        rows = ring and AR == 4
        assert NCV - work >= 14, (T, D, NF, NCV, AR)
        clob = ["v%d" % n for n in range(NCV - work, NCV + FO + NF * T)] + ["vcc", "scc", "m0", "memory"]
        clob += ["s%d" % n for n in [58, 59] + list(range(64, 76)) + [79, 80, 81, 99]]
        if AR in (0, 4):
            clob += ["s%d" % n for n in range(24, 56)]
        if ring:
            clob += ["s%d" % n for n in range(ring_base(AR), ring_base(AR) + 16)]
        core_lines = []
        core_lines.append("template <> struct Core<%d, %d, %d, %d, %d> {" % core)
        core_lines.append("    // runs one unit: its tile is loaded, then its programs run to their partial sums (or outputs);")
        core_lines.append("    // with `probe` only the address of the handler table is returned")
        core_lines.append("    static __device__ __forceinline__ void run(const CoreUnit& u, uint32_t probe, uint64_t& table) {")
        core_lines.append("#ifdef __HIP_DEVICE_COMPILE__")
        core_lines.append("        uint32_t off = u.off, end = u.end, kind = u.kind;")
        if rows:
            core_lines.append("        uint32_t own_kind = u.own_kind;")
        core_lines.append('        asm volatile("%s"' % text)
        core_lines.append('            : "+{s62}"(off), "+{s96}"(end), "+{s93}"(kind), "={s[76:77]}"(table)'
                          + (', "+{s98}"(own_kind)' if rows else ''))
        ins = [("s[60:61]", "u.code"), ("s63", "probe"), ("s78", "u.burst"), ("s[82:83]", "u.X"), ("s[84:85]", "u.stride"),
               ("s86", "u.n_load"), ("s87", "u.left"), ("s[88:89]", "u.y"), ("s[90:91]", "u.partials"),
               ("s92", "u.part_stride"), ("s[94:95]", "u.cases"), ("s97", "u.lds_y")]
        if rows:
            ins += [("s56", "u.own_off"), ("s57", "u.own_end")]
        if AR == 2:
            ins.append(("s98", "u.bits"))
        if AR in (0, 4):
            ins.append(("s[100:101]", "u.coef"))
        core_lines.append("            : " + ", ".join('"{%s}"(%s)' % i for i in ins))
        core_lines.append("            : " + ", ".join('"%s"' % x for x in clob) + ");")
        core_lines.append("#endif")
        core_lines.append("    }")
        core_lines.append("};")
        cores.append(core_lines)
        host.append((T, D, NF, NCV, AR, hs_tag, hs, nslots, ring))
    lines.append("")
    lines.append("struct CoreHandlerKey { uint8_t kind, op; int8_t p1, p2; };")
    done = set()
    for (T, D, NF, NCV, AR, tag, hs, nslots, ring) in host:
        if tag in done:
            continue
        done.add(tag)
        lines.append("static const CoreHandlerKey kCoreKeys_%s[] = {" % tag)
        lines.append("    " + ", ".join("{%d,%d,%d,%d}" % (h.kind, h.op, h.p1, h.p2) for h in hs))
        lines.append("};")
        lines.append("static const uint16_t kCoreSlots_%s[] = {" % tag)
        lines.append("    " + ", ".join(str(h.slot) for h in hs))
        lines.append("};")
    lines.append("struct CoreVariantDesc { int t, d, nf, ncv, arith; const CoreHandlerKey* keys; const uint16_t* slots; "
                 "int n; int slot_bytes; int xx; bool ring; "
                 "int waves, rows_base, cap; bool by_number_only; };")
    lines.append("// xx: levels with one-pass handlers of two variables; waves: waves of a block; rows_base: LDS address of its rows, or 0;")
    lines.append("// cap: features it takes (more than nf: the others in LDS); by_number_only: never chosen by default")
    lines.append("static const CoreVariantDesc kCoreVariants[] = {")
    for (T, D, NF, NCV, AR, tag, hs, nslots, ring) in host:
        lines.append("    {%d, %d, %d, %d, %d, kCoreKeys_%s, kCoreSlots_%s, %d, %d, %d, %s, %d, %d, %d, %s},"
                     % (T, D, NF, NCV, AR, tag, tag, len(hs), RING_SLOT if ring else SLOT, xx_levels(D, NF, AR, ring),
                        "true" if ring else "false", waves_per_block(T, D, NF, NCV, AR, ring),
                        rows_base(T, D, NF, NCV, AR) if ring and AR == 4 else 0,
                        WIDE.get((T, D, NF, NCV, AR), NF) if ring else NF,
                        "true" if (T, D, NF, NCV, AR) in BY_NUMBER_ONLY else "false"))
    lines.append("};")
    path = os.path.join(out_dir, "core_gen.inc")
    write_if_changed(path, "\n".join(lines) + "\n")
    # one translation unit per kernel variant, and the launch table
    disp = ["// Generated by gen_core.py -- do not edit.", "#pragma once", "",
            "typedef hipError_t (*CoreLaunchFn)(const CoreArgs&, uint32_t, hipStream_t);",
            "typedef int (*CoreOccupancyFn)();"]
    for core_lines, (T, D, NF, NCV, AR, tag, hs, nslots, ring) in zip(cores, host):
        name = vname((T, D, NF, NCV, AR))
        W = waves_per_block(T, D, NF, NCV, AR, ring)
        disp.append("hipError_t core_launch_%s(const CoreArgs& a, uint32_t blocks, hipStream_t s);" % name)
        disp.append("int core_occupancy_%s();" % name)
        tu = ["// Generated by gen_core.py -- do not edit.  Kernel variant %s." % tag,
              '#include "core_body.h"', "", "namespace gpx {"] + core_lines + ["",
              "GPX_KERNEL(%d, %d, %d, %d, %d, %d, %s, %s)" % (T, D, NF, NCV, AR, W, "true" if ring and AR == 4 else "false", name), "",
              "hipError_t core_launch_%s(const CoreArgs& a, uint32_t blocks, hipStream_t s) {" % name,
              "    hipLaunchKernelGGL(k_core_%s, dim3(blocks), dim3(a.direct ? 64u * (uint32_t)a.direct : %du), (uint32_t)a.n_rows * %du, s, a);"
              % (name, 64 * W, 256 * T),
              "    return hipGetLastError();", "}", "",
              "int core_occupancy_%s() {" % name,
              "    int n = 0;",
              "    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_core_%s, %d, 0) != hipSuccess) n = 1;" % (name, 64 * W),
              "    return n;", "}", "}  // namespace gpx", ""]
        write_if_changed(os.path.join(out_dir, "core_v_%s.hip" % name), "\n".join(tu))
    names = [vname(h[:5]) for h in host]
    disp.append("static const CoreLaunchFn kCoreLaunch[] = {%s};" % ", ".join("core_launch_" + n for n in names))
    disp.append("static const CoreOccupancyFn kCoreOccupancy[] = {%s};"
                % ", ".join("core_occupancy_" + n for n in names))
    write_if_changed(os.path.join(out_dir, "core_dispatch.inc"), "\n".join(disp) + "\n")
    for (T, D, NF, NCV, AR, tag, hs, nslots, ring) in host:
        print("%s%s: %d handlers, %d slots (%d KiB)" % (tag, "a" if AR == 1 else "", len(hs), nslots, nslots * (RING_SLOT if ring else SLOT) // 1024))
    return path


def variant_sources():
    """File names of the generated per-variant translation units."""
    return ["core_v_%s.hip" % vname(v) for v in VARIANTS + RING_VARIANTS]


def write_if_changed(path, text):
    """Write text unless the file already holds it (keeps mtimes for incremental builds)."""
    if os.path.exists(path):
        with open(path) as f:
            if f.read() == text:
                return
    with open(path + ".tmp", "w") as f:
        f.write(text)
    os.replace(path + ".tmp", path)


if __name__ == "__main__":
    main(sys.argv[1] if len(sys.argv) > 1 else ".")
