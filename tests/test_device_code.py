"""The waits around inline assembly in the gfx950 code of this package (compiled here to assembly, no GPU).

The compiler puts the wait states that the hardware asks for between its own instructions, but it does not look
into inline assembly: an instruction there can read a register before the result is in it.  These tests follow
every path through the assembly and check each pair of a writer and a reader of which at least one is inline."""
import concurrent.futures
import os
import re
import subprocess

import pytest

from paper_2509_10918_amd import build

# wait states that the compiler leaves between its own instructions (read off small kernels compiled with it):
# kind of writer -> kind of reader.  Products differ by their size; 19 is the longest.
NEEDED = {
    ("product", "vector"): 19,   # matrix product -> vector instruction that reads the result
    ("product", "lane"): 19,
    ("scalar", "vector"): 2,     # vector instruction that writes a scalar register -> vector instruction that reads it
    ("scalar", "memory"): 5,     # -> load or store that takes its address from it
    ("vector", "lane"): 2,       # vector instruction -> row moves of the result between lanes, reads of single lanes
    ("slow", "vector"): 1,       # exponential, root, reciprocal -> vector instruction that reads the result
    ("slow", "lane"): 2,
}
HORIZON = 24


def _regs(text, kind):
    out = set()
    for one, lo, hi in re.findall(r"(?<![\w.])%s(?:(\d+)\b|\[(\d+):(\d+)\])" % kind, text):
        out.update((int(one),) if one else range(int(lo), int(hi) + 1))
    return {(kind, r) for r in out}


class Instr:
    __slots__ = ("op", "inline", "line", "waits", "reads", "writes", "write_kind", "read_kind")

    def __init__(self, text, inline, line):
        op, _, rest = text.partition(" ")
        ops = re.findall(r"[^,\[]+(?:\[[^\]]*\])?", rest)
        self.op, self.inline, self.line = op, inline, line
        self.waits = int(ops[0], 0) + 1 if op == "s_nop" else 1
        vector = op.startswith("v_")
        memory = op.startswith(("ds_", "global_", "buffer_", "flat_", "scratch_"))
        n_out = 1 if vector or (memory and ("load" in op or "read" in op) and "lds" not in op) else 0
        if op.startswith(("s_load", "s_mov", "s_add", "s_sub", "s_and", "s_or", "s_lsh", "s_mul", "s_ff1", "s_cselect", "s_min",
                          "s_max", "s_bfe", "s_lshr", "s_ashr", "s_xor", "s_not", "s_andn2", "s_bcnt")):
            n_out = 1
        if op.startswith(("v_add_co", "v_sub_co", "v_addc", "v_subb", "v_div_scale", "v_mad_u64", "v_mad_i64")):
            n_out = 2
        out, ins = ops[:n_out], ops[n_out:]
        if "swap" in op:
            out = ins = ops
        # (an accumulator may live in the a registers: the other half of the same file)
        self.writes = set().union(*(_regs(o, k) for o in out for k in "vas"), set())
        self.reads = set().union(*(_regs(o, k) for o in ins for k in "vas"), set())
        if op.startswith("v_") and "vcc" in rest:
            (self.writes if any("vcc" in o for o in out) else self.reads).add(("s", "vcc"))
        self.write_kind = self.read_kind = None
        if vector:
            self.write_kind = ("product" if op.startswith(("v_mfma", "v_smfma")) else
                               "slow" if re.match(r"v_(exp|log|rcp|rsq|sqrt|sin|cos)_", op) else "vector")
            moves = "quad_perm" in rest or "row_" in rest or "permlane" in op or "readlane" in op or "readfirstlane" in op
            self.read_kind = "lane" if moves else "vector"
        elif memory:
            self.read_kind = "memory"

    def kind_of(self, reg):
        """Kind of this instruction as the writer of `reg` (scalar registers: by a vector instruction only)."""
        if reg[0] == "s":
            return "scalar" if self.op.startswith("v_") else None
        return self.write_kind


def _functions(path):
    """(name, blocks): blocks as (instructions, labels of the blocks that may follow)."""
    name, blocks, labels, cur, inline = None, [], {}, [], False
    for number, raw in enumerate(open(path), 1):
        text = raw.strip()
        if text.startswith(";;#ASM"):
            inline = text.startswith(";;#ASMSTART")
            continue
        text = text.split(";")[0].strip()
        m = re.match(r"([\w.$]+):$", text)
        if m and m.group(1).startswith("_Z"):
            name, blocks, labels, cur = m.group(1), [], {}, []
            continue
        if name is None:
            continue
        if text.startswith(".Lfunc_end"):
            blocks.append((cur, []))
            yield name, blocks, labels
            name = None
        elif m:  # a label begins a block that the one before may run into
            blocks.append((cur, [len(blocks) + 1]))
            cur = []
            labels[m.group(1)] = len(blocks)
        elif text and not text.startswith("."):
            ins = Instr(text, inline, number)
            cur.append(ins)
            if ins.op.startswith("s_cbranch"):
                blocks.append((cur, [len(blocks) + 1, text.split()[1]]))
                cur = []
            elif ins.op == "s_branch":
                blocks.append((cur, [text.split()[1]]))
                cur = []
            elif ins.op in ("s_endpgm", "s_setpc_b64"):
                blocks.append((cur, []))
                cur = []


def short_waits(path):
    """Readers (function, line of the assembly, text) that come too early after their writer on some path."""
    found = set()
    for name, blocks, labels in _functions(path):
        if not any(i.inline for b, _ in blocks for i in b):
            continue
        # state: (register, kind of writer, was it inline) -> wait states since
        entry = [{} for _ in blocks]
        todo, seen = list(range(len(blocks))), [False] * len(blocks)
        while todo:
            n = todo.pop()
            seen[n] = True
            state = dict(entry[n])
            for ins in blocks[n][0]:
                if ins.read_kind and state:
                    for (reg, kind, was_inline), age in state.items():
                        if reg in ins.reads and (ins.inline or was_inline) and age < NEEDED.get((kind, ins.read_kind), 0):
                            found.add((name, ins.line, f"{ins.op} after {age} of {NEEDED[kind, ins.read_kind]} wait states"))
                state = {k: a + ins.waits for k, a in state.items() if k[0] not in ins.writes and a + ins.waits < HORIZON}
                # (the age counts from the writer itself: the next instruction sees 0)
                state.update({(r, ins.kind_of(r), ins.inline): 0 for r in ins.writes if ins.kind_of(r)})
            for nxt in blocks[n][1]:
                nxt = labels.get(nxt) if isinstance(nxt, str) else nxt
                if nxt is None or nxt >= len(blocks):
                    continue
                lower = {k: a for k, a in state.items() if a < entry[nxt].get(k, HORIZON)}
                if lower:
                    entry[nxt].update(lower)
                    todo.append(nxt)
    return sorted(found)


def _scan(tmp_path, body):
    path = tmp_path / "k.s"
    path.write_text("_Zk:\n" + body + "\n.Lfunc_end0:\n")
    return short_waits(path)


PRODUCT = "v_mfma_f32_16x16x32_bf16 v[4:7], v[8:11], v[12:15], 0\n"


def _inline(text):
    return f";;#ASMSTART\n{text}\n;;#ASMEND\n"


@pytest.mark.parametrize("body,early", [
    (PRODUCT + "s_nop 7\n" + _inline("v_max3_f32 v1, v4, v5, v6"), True),
    (PRODUCT + "s_nop 7\ns_nop 7\ns_nop 2\n" + _inline("v_max3_f32 v1, v4, v5, v6"), False),
    (PRODUCT + "v_max3_f32 v1, v4, v5, v6\n", False),                                  # the compiler's own: its affair
    (PRODUCT + _inline("v_max3_f32 v4, v1, v2, v3"), False),                           # writes, does not read
    (PRODUCT + "v_mov_b32 v4, v1\n" + _inline("v_max_f32 v1, v4, v2"), False),         # another result by then
    # the branch around the masking of the last tile: long on one path, short on the other
    (PRODUCT + "s_cbranch_scc1 .L1\n" + "s_nop 15\ns_nop 15\n.L1:\n" + _inline("v_max_f32 v1, v7, v2"), True),
    ("v_readlane_b32 s4, v1, s9\ns_mov_b32 s5, 0\n" + _inline("v_mov_b32 v2, s4"), True),
    ("v_readlane_b32 s4, v1, s9\ns_nop 1\n" + _inline("v_mov_b32 v2, s4"), False),
    ("v_readlane_b32 s4, v1, s9\ns_mov_b32 s4, 0\n" + _inline("v_mov_b32 v2, s4"), False),   # scalar unit: no wait
    ("v_readfirstlane_b32 s4, v1\ns_nop 1\n" + _inline("global_load_dwordx4 v[4:7], v2, s[4:5]"), True),
    (_inline("v_mov_b32 v1, v2") + "s_nop 0\nv_mov_b32_dpp v3, v1 quad_perm:[1,0,3,2]\n", True),
    ("v_exp_f32 v1, v2\n" + _inline("v_add_f32 v3, v1, v1"), True),
    # round a loop
    (".L1:\n" + _inline("v_max_f32 v1, v7, v2") + PRODUCT + "s_cbranch_scc1 .L1\n", True),
])
def test_the_scan_itself(tmp_path, body, early):
    assert bool(_scan(tmp_path, body)) == early


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    where = tmp_path_factory.mktemp("asm")

    def one(src):
        out = str(where / (src + ".s"))
        subprocess.run(["hipcc", *build.FLAGS, "-S", "--offload-device-only", os.path.join(build.CSRC, src), "-o", out],
                       check=True, capture_output=True)
        return out
    with concurrent.futures.ThreadPoolExecutor(8) as pool:
        return dict(zip(build.SOURCES, pool.map(one, build.SOURCES)))


@pytest.mark.parametrize("src", build.SOURCES)
def test_inline_assembly_waits_for_its_operands(assembly, src):
    early = short_waits(assembly[src])
    assert not early, "\n".join(map(str, early[:20]))
