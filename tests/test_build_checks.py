"""Static checks of generated code (CPU only; need hipcc, which cross-compiles without a GPU).

The W8A8 product writes each accumulation chain (four MFMAs, the first taking its C operand as an
inline constant the compiler would otherwise hold in 16 registers) as ONE assembly statement, so the
chain accumulates in place by construction.  The compiler does not know the statement holds matrix
products and inserts no wait states before a vector instruction that reads the chain's result (the
hardware does not interlock that case); the kernel is written so that every such reader comes a
whole chain later in program order.  The first test compiles the kernel to assembly and checks both: the
chains are in place, and at least 18 instructions (the wait states the longest case needs) lie
between the end of a chain and the first instruction that reads its result.

The second test follows every path behind every matrix product written in assembly, in all sources that have
them: nothing reads OR writes the product's result before it has landed, branches and loops included.

The third holds every kernel to its registers: a reload from scratch memory waits for every load in flight, the ones a
kernel has just requested ahead included."""
import functools
import os
import re
import shutil
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_16093_amd", "csrc")


def _hipcc():
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    return None


def _regs(operand_text):
    """Register numbers named in an operand string: v12 and v[12:15] forms."""
    regs = set()
    for a, b in re.findall(r"\bv\[(\d+):(\d+)\]", operand_text):
        regs.update(range(int(a), int(b) + 1))
    regs.update(int(x) for x in re.findall(r"\bv(\d+)\b", operand_text))
    return regs


@functools.lru_cache(maxsize=None)
def _assembly(source):
    from paper_2512_16093_amd import build as b
    src = os.path.join(CSRC, source)
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "k.s")
        flags = [f for f in b.FLAGS if f not in ("-fPIC",)]
        r = subprocess.run([_hipcc()] + flags + ["-S", "--cuda-device-only", src, "-o", out],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        return open(out).read()


@pytest.mark.skipif(_hipcc() is None, reason="hipcc not available")
def test_w8a8_chains_are_in_place_and_read_late_enough():
    text = _assembly("k_w8a8.hip")
    # instructions only (no labels, directives, comments)
    ins = [l.split(";")[0].strip() for l in text.splitlines()]
    ins = [l for l in ins if l and not l.startswith(".") and not l.endswith(":") and re.match(r"[a-z]", l)]
    pat = re.compile(r"v_mfma_i32_32x32x32_i8 (v\[(\d+):(\d+)\]), v\[\d+:\d+\], v\[\d+:\d+\], (\S+)")
    starts = [i for i, l in enumerate(ins) if l.startswith("v_mfma_i32_32x32x32_i8") and l.endswith("0.15915494")]
    assert len(starts) >= 8, "expected the chains' first MFMAs to take the inline constant"
    for i in starts:
        m0 = pat.match(ins[i])
        dst, lo, hi = m0.group(1), int(m0.group(2)), int(m0.group(3))
        mine = set(range(lo, hi + 1))
        # the chain: the next three matrix products that write these registers accumulate in place
        steps, last = 0, i
        for d, l in enumerate(ins[i + 1:i + 200]):
            m = pat.match(l)
            if m and m.group(1) == dst:
                assert m.group(4) == dst, (ins[i], l)
                steps, last = steps + 1, i + 1 + d
                if steps == 3:
                    break
        assert steps == 3, ins[i]
        # the first instruction that reads the result: at least 18 wait states behind the chain's last product
        # (a matrix product that has to wait for its own chain counts as 8, s_nop n as n + 1, anything else as 1)
        waited = 0
        for l in ins[last + 1:last + 400]:
            if l.startswith("s_endpgm"):
                break
            operands = l.split(None, 1)[1] if " " in l else ""
            srcs = operands.split(",", 1)[1] if "," in operands else ""     # everything after the destination
            if _regs(srcs) & mine:
                assert waited >= 18, (ins[i], l, "result read after only %d wait states" % waited)
                break
            if _regs(operands.split(",", 1)[0]) & mine:
                break                            # overwritten before any read (how late: the next test)
            nop = re.match(r"s_nop (\d+)", l)
            waited += int(nop.group(1)) + 1 if nop else (8 if l.startswith("v_mfma") and l.split(",")[-1].strip().startswith("v[") else 1)


# ---- every access behind an assembly product, on every path
PASSES = 8    # wait states a 32 x 32 product of either kind occupies the matrix pipe: the next one is issued behind them
LANDED = 12   # wait states before another instruction may touch its result (gfx950; the compiler puts `s_nop 11` behind its own)
OPERANDS = 2  # wait states between a vector instruction's result and a product that takes it as an operand


class _Ins:
    def __init__(self, text, in_asm):
        self.text, self.op = text, text.split()[0]
        operands = [o.strip() for o in re.split(r",(?![^\[]*\])", text[len(self.op):])]
        self.operands, self.in_asm, self.asm_product = operands, in_asm, in_asm and self.op.startswith("v_mfma")
        self.product = self.op.startswith("v_mfma")
        self.all = _files(" ".join(operands))
        self.first, self.rest = _files(operands[0]), _files(" ".join(operands[1:]))
        self.states = int(operands[0]) + 1 if self.op == "s_nop" else 1


def _files(text):
    """Registers named in an operand string, with their file: ("v", 12), ("a", 3)."""
    regs = set()
    for f, lo, hi in re.findall(r"\b([va])\[(\d+):(\d+)\]", text):
        regs.update((f, x) for x in range(int(lo), int(hi) + 1))
    regs.update((f, int(x)) for f, x in re.findall(r"\b([va])(\d+)\b", text))
    return frozenset(regs)


def _kernels(text):
    """Mangled name -> (instructions, label -> index of the instruction behind it)."""
    kernels, cur, in_asm = {}, None, False
    for line in text.splitlines():
        name, label = re.match(r"(_Z\w+):", line), re.match(r"(\.LBB\w+):", line)
        if name:
            cur = kernels.setdefault(name.group(1), ([], {}))
        elif label and cur:
            cur[1][label.group(1)] = len(cur[0])
        in_asm = (in_asm or "#ASMSTART" in line) and "#ASMEND" not in line
        ins = line.split(";")[0].strip()
        if cur and re.match(r"[a-z]\w*(\s|$)", ins):
            cur[0].append(_Ins(ins, in_asm))
    return kernels


def _next(ins, labels, x):
    op = ins[x].op
    if op == "s_endpgm":
        return []
    if op == "s_branch":
        return [labels[ins[x].operands[0]]]
    return [labels[ins[x].operands[0]], x + 1] if op.startswith("s_cbranch") else [x + 1]


def _early_accesses(ins, labels):
    """(assembly products, [product, instruction that touches its result too early, wait states between])."""
    products, found = 0, []
    for x, p in enumerate(ins):
        if not p.asm_product:
            continue
        products += 1
        todo, seen = [(y, 1, PASSES) for y in _next(ins, labels, x)], set()   # (instruction, its time, when the pipe is free)
        while todo:
            y, t, free = todo.pop()
            if (y, t, free) in seen:
                continue
            seen.add((y, t, free))
            i = ins[y]
            if i.product:
                t = max(t, free)
                free = t + PASSES
            if t > LANDED:
                continue
            if i.all & p.first:
                # the chain goes on in place (or starts again in the same registers): the hardware holds that back
                if not (i.product and i.first == p.first and not _files(" ".join(i.operands[1:3])) & p.first):
                    found.append((p.text, i.text, t - 1))
                continue
            todo += [(z, t + i.states, free) for z in _next(ins, labels, y)]
    return products, found


def _late_operands(ins, labels):
    """[vector instruction, assembly product that takes its result too early, wait states between]."""
    found = []
    for x, p in enumerate(ins):
        if not p.op.startswith("v_") or p.product:
            continue
        todo = [(y, 0) for y in _next(ins, labels, x)]
        while todo:
            y, t = todo.pop()
            if t >= OPERANDS:
                continue
            if ins[y].asm_product and ins[y].rest & p.first:
                found.append((p.text, ins[y].text, t))
            else:
                todo += [(z, t + ins[y].states) for z in _next(ins, labels, y)]
    return found


# kernel -> instances and assembly products of each: the dQ kernel forms S and dP of a prologue and two steps, QT tiles of
# eight products each; dK/dV (one key block) S and dP of two tiles in two steps; W8A8 chains of four per output tile
EXPECTED = {
    "k_bwd.hip": {r"bwd_dq_kernelILi\dELi1": (4, 48), r"bwd_dq_kernelILi\dELi2": (4, 96), r"bwd_dkv_kernelILi1": (6, 64),
                  r"bwd_dq_dkv_kernel": (6, 64 + 48)},
    "k_w8a8.hip": {r"w8a8_gemm_kernelE": (1, 96), r"w8a8_gemm_splitk_kernelILi2ELi2": (3, 16),
                   r"w8a8_gemm_splitk_kernelILi1ELi2": (2, 8), r"w8a8_gemm_splitk_kernelILi1ELi1": (2, 4),
                   r"w8a8_gemm_wide_kernelILi2ELi3": (1, 48), r"w8a8_gemm_wide_kernelILi2ELi4": (2, 64),
                   r"w8a8_gemm_wide_kernelILi2ELi5": (2, 80), r"w8a8_gemm_wide_kernelILi4ELi3": (2, 96)},
}


@pytest.mark.skipif(_hipcc() is None, reason="hipcc not available")
@pytest.mark.parametrize("source", sorted(EXPECTED))
def test_products_have_landed_before_anything_touches_them(source):
    counts = {}
    for name, (ins, labels) in _kernels(_assembly(source)).items():
        products, early = _early_accesses(ins, labels)
        assert not early, (name, early[:4])
        assert not _late_operands(ins, labels), (name, _late_operands(ins, labels)[:4])
        if products:
            counts[name] = products
    for pattern, (instances, products) in EXPECTED[source].items():
        mine = [n for k, n in counts.items() if re.search(pattern, k)]
        assert mine == [products] * instances, (pattern, mine)
    assert len(counts) == sum(n for n, _ in EXPECTED[source].values()), sorted(counts)


# ---- assembly that switches lanes off and, behind its copies, all of them on: it may stand only where all of them are on
def _scalars(operand):
    m = re.match(r"s\[(\d+):(\d+)\]$", operand) or re.match(r"s(\d+)$", operand)
    return range(int(m.group(1)), int(m.group(m.lastindex)) + 1) if m else range(106, 108) if operand == "vcc" else range(0)


def _narrowed(ins, labels):
    """(assembly writes of exec from a register, those of them that some path reaches with a lane switched off).  Known along
    every path: are all lanes on, and which scalar registers hold a mask of all of them (halves of pairs; `lane` names a
    vector register's lane, where the compiler parks scalar registers)."""
    state, todo, writes, found = {0: (True, frozenset())}, [0], set(), set()
    while todo:
        x = todo.pop()
        full, masks = state[x]
        i = ins[x]
        op, o = i.op, i.operands
        holds = lambda name: full if name == "exec" else name == "-1" or (len(_scalars(name)) == 2 and masks.issuperset(_scalars(name)))
        if i.in_asm and o[0] == "exec" and o[1] != "-1":
            writes.add(x)
            if not full:
                found.add(x)
        after, parked = full, masks
        if op in ("s_and_saveexec_b64", "s_andn2_saveexec_b64", "s_or_saveexec_b64"):
            after = op.startswith("s_or") and (full or holds(o[1]))
            parked = masks - set(_scalars(o[0])) | (set(_scalars(o[0])) if full else set())
        elif o[0] == "exec":
            after = {"s_mov_b64": holds(o[1]), "s_or_b64": any(holds(y) for y in o[1:])}.get(op, False)
        elif op == "s_mov_b64":
            parked = masks - set(_scalars(o[0])) | (set(_scalars(o[0])) if holds(o[1]) else set())
        elif op in ("v_writelane_b32", "v_readlane_b32"):
            lane = lambda v, l: ("lane", v, l)
            gone, source = ({lane(o[0], o[2])}, set(_scalars(o[1]))) if op[2] == "w" else (set(_scalars(o[0])), {lane(o[1], o[2])})
            parked = masks - gone | (gone if source and masks >= source else set())
        elif not op.startswith(("s_cbranch", "s_branch", "s_cmp", "s_bitcmp", "s_waitcnt", "s_nop", "s_barrier", "global_load", "ds_")):
            parked = masks - set(_scalars(o[0])) - set(_scalars(o[1]) if len(o) > 1 and op.startswith("v_") else ())
        for y in _next(ins, labels, x):
            old = state.get(y)
            new = (after, parked) if old is None else (after and old[0], parked & old[1])
            if new != old:
                state[y] = new
                todo.append(y)
    return len(writes), [ins[x].text for x in sorted(found)]


@pytest.mark.skipif(_hipcc() is None, reason="hipcc not available")
def test_copies_of_some_lanes_stand_where_all_lanes_are_on():
    writes = {}
    for name, (ins, labels) in _kernels(_assembly("k_bwd.hip")).items():
        n, found = _narrowed(ins, labels)
        assert not found, (name, found[:4])
        if n:
            writes[re.match(r"_ZN3sla\d+(\w+?)I", name).group(1)] = writes.get(re.match(r"_ZN3sla\d+(\w+?)I", name).group(1), 0) + 1
    assert writes == {"bwd_dq_kernel": 8, "bwd_dkv_kernel": 6, "bwd_dq_dkv_kernel": 6}, writes


def test_the_check_of_lanes_sees_what_it_is_for():
    copies = "\t;;#ASMSTART\n\ts_mov_b64 exec, s[4:5]\n\ts_mov_b64 exec, -1\n\t;;#ASMEND\n"

    def found(body):
        (ins, labels), = _kernels("_Zk:\n" + body + "\ts_endpgm\n").values()
        n, bad = _narrowed(ins, labels)
        assert n == 1
        return len(bad)
    branch = "\ts_and_saveexec_b64 s[0:1], vcc\n\ts_cbranch_execz .LBB0_1\n%s.LBB0_1:\n\ts_or_b64 exec, exec, s[0:1]\n%s"
    assert found(copies) == found(branch % ("", copies)) == 0
    assert found(branch % (copies, "")) == found("\ts_mov_b32 s0, 0\n" + copies.join(("\ts_and_b64 exec, exec, vcc\n", ""))) == 1
    assert found(branch % ("\ts_mov_b32 s1, s2\n", copies)) == 1      # (the saved mask is gone)
    assert found(branch % ("\tv_writelane_b32 v9, s0, 3\n\tv_writelane_b32 v9, s1, 4\n\ts_mov_b64 s[0:1], 0\n"
                           "\tv_readlane_b32 s0, v9, 3\n\tv_readlane_b32 s1, v9, 4\n", copies)) == 0
    assert found(".LBB0_1:\n" + copies + "\ts_andn2_b64 exec, exec, s[6:7]\n\ts_cbranch_execnz .LBB0_1\n") == 1


# The selection of rows beyond 6144 key blocks indexes an array that does not fit the registers.
SCRATCH_BY_DESIGN = r"select_kernelILi128E"


@pytest.mark.skipif(_hipcc() is None, reason="hipcc not available")
@pytest.mark.parametrize("source", sorted(f for f in os.listdir(CSRC) if f.startswith("k_") and f.endswith(".hip")))
def test_no_kernel_keeps_registers_in_scratch_memory(source):
    """What the compiler reports of every kernel: bytes of scratch memory per lane, and vector registers spilled to it."""
    text = _assembly(source)
    kernels = re.findall(r"\.private_segment_fixed_size: (\d+)(?:(?!\.symbol).)*\.symbol: +(\S+)\.kd(?:(?!\.private_segment).)*"
                         r"\.vgpr_spill_count: (\d+)", text, re.S)
    assert len(kernels) == len(re.findall(r"^\s*\.amdhsa_kernel ", text, re.M)) > 0
    held = [(name, scratch, spilled) for scratch, name, spilled in kernels
            if (scratch, spilled) != ("0", "0") and not re.search(SCRATCH_BY_DESIGN, name)]
    assert not held, held


def test_every_source_with_assembly_products_is_checked():
    assert {f for f in os.listdir(CSRC) if 'asm volatile("v_mfma' in open(os.path.join(CSRC, f)).read()} == set(EXPECTED)


def test_the_check_sees_what_it_is_for():
    """Planted code: a result read one product later, one overwritten behind a taken branch, one past a loop's back edge."""
    product = "\t;;#ASMSTART\n\tv_mfma_f32_32x32x16_bf16 v[0:15], v[20:23], a[0:3], 0\n\t;;#ASMEND\n"
    other = product.replace("v[0:15]", "v[32:47]")

    def early(body):
        (ins, labels), = _kernels("_Zk:\n" + body + "\ts_endpgm\n").values()
        return len(_early_accesses(ins, labels)[1])
    read, write = "\tv_add_f32_e32 v50, v3, v51\n", "\tv_mov_b32_e32 v4, v50\n"
    assert early(product + read) == early(product + write) == early(product + other + read) == 1
    assert early(product + other + other + read) == 0 and early(product + "\ts_nop 11\n" + read) == 0
    assert early(product + "\ts_nop 10\n" + write) == 1
    assert early(product + "\ts_cbranch_scc1 .LBB0_1\n\ts_nop 15\n" + read + ".LBB0_1:\n" + write) == 1
    assert early(".LBB0_1:\n" + write + product + "\ts_cbranch_scc0 .LBB0_1\n\ts_nop 15\n") == 1
    assert early(product + product.replace("a[0:3], 0", "a[0:3], v[0:15]") + "\ts_nop 15\n" + read) == 0
    (ins, labels), = _kernels("_Zk:\n\tv_mov_b32_e32 v21, v50\n\ts_nop 0\n" + product + "\ts_endpgm\n").values()
    assert len(_late_operands(ins, labels)) == 1
