"""Distances that inline assembly has to keep by itself, along every path of the compiled kernels (no GPU).

The compiler puts wait states between its own instructions; it sees neither into a block of inline assembly nor what reads the block's
results.  Checked on the assembly of the sources that have such blocks, over their control flow: backwards from each
instruction through every predecessor, loops and skipped blocks included."""
import functools
import os
import re
import subprocess

import pytest

from paper_2602_04789_amd import build as B

SOURCES = ["lf_attn.hip", "lf_attn_wide.hip", "lf_attn_bwd.hip", "lf_attn_bwd_wide.hip", "lf_attn_bwd_q_wide.hip"]
FAR = 11       # the longest distance asked for, in wait states


class Instr:
    def __init__(self, text):
        self.text, self.before = text, []
        self.op, _, rest = text.partition(" ")
        args = [x.strip() for x in re.split(r",\s*(?![^\[]*\])", rest.strip())]
        self.product = "mfma" in self.op
        self.vector = self.op.startswith("v_") and not self.product
        self.memory = self.op.startswith(("buffer_", "global_", "flat_", "scratch_"))
        self.states = int(args[0], 0) + 1 if self.op == "s_nop" else 1
        self.passes = 0 if not self.product else 2 if "4x4x4" in self.op else 8
        stores = self.op.startswith(("ds_write", "ds_add", "buffer_store", "global_store", "scratch_store", "flat_store")) or "lds" in args[-1].split()
        self.written, self.read = set(), registers(rest)
        if self.product or (self.op.startswith(("v_", "s_", "ds_read", "buffer_load", "global_load", "scratch_load")) and not stores):
            n = 2 if "swap" in self.op else 1
            self.written = registers(" ".join(args[:n]))
            self.read = registers(" ".join(args if "swap" in self.op or "dot2c" in self.op or "fmac" in self.op else args[1:]))
        if self.op.startswith(("s_cmp", "s_bitcmp")):
            self.written, self.read = {("scc", 0)}, registers(rest)
        self.sources = [registers(x) for x in args[1:4]] if self.product else []
        self.transcendental = re.match(r"v_(exp|log|rcp|rsq|sqrt|sin|cos)_", self.op) is not None
        self.m0 = self.op.startswith("s_") and args[0] == "m0"


def registers(text):
    out = set()
    for m in re.finditer(r"\b([vas])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        first, last = (m[2], m[3]) if m[2] else (m[4], m[4])
        out |= {(m[1], i) for i in range(int(first), int(last) + 1)}
    return out | ({("vcc", 0)} if re.search(r"\bvcc\b", text) else set())


def program(lines):
    """Instructions with their predecessors (`before`)."""
    code, labels, open_ends, jumps = [], {}, [], []
    for line in lines:
        line = line.split(";")[0].split("//")[0].strip()
        m = re.match(r"([.\w]+):", line)
        if m:
            labels[m[1]] = len(code)
            if not m[1].startswith(".L"):
                open_ends = []                       # a new kernel
            continue
        if not re.match(r"(s|v|ds|buffer|global|flat|scratch)_\w+", line):
            continue
        x = Instr(line)
        x.before += open_ends
        code.append(x)
        m = re.match(r"s_(c?)branch\w*\s+(\.LBB\w+)", line)
        if m:
            jumps.append((x, m[2]))
        open_ends = [] if line.startswith("s_endpgm") or (m and not m[1]) else [x]
    for x, label in jumps:
        if labels[label] < len(code):
            code[labels[label]].before.append(x)
    return code


def stall(x, seen={}):
    """Wait states that a product stands before it issues, itself among them: the unit takes one at a time.  The least of all paths."""
    key = id(x)
    if key not in seen:
        best = 8
        todo = [(p, 0) for p in x.before]
        while todo:
            p, since = todo.pop()
            if p.product or since >= 8 or not p.before:
                best = min(best, max(1, p.passes - since))
            else:
                todo += [(q, since + p.states) for q in p.before]
        seen[key] = (x, best)        # (x kept: its id stays its own)
    return seen[key][1]


def hazards(lines):
    found = set()
    for x in program(lines):
        # registers that a nearer instruction has written do not count for what lies behind it
        todo, visited = [(p, 0, frozenset()) for p in x.before], set()
        while todo:
            p, since, hidden = todo.pop()
            if since >= FAR or (id(p), since, hidden) in visited:
                continue
            visited.add((id(p), since, hidden))
            made = p.written - hidden
            scalars = {r for r in made if r[0] in ("s", "vcc")}
            need = 0
            if p.vector and x.memory and scalars & x.read:
                need = 5
            if p.vector and x.vector and scalars & x.read:
                need = max(need, 2)
            if p.vector and "lane" in x.op and x.vector and p.written & x.read - scalars:
                need = max(need, 1)
            if p.transcendental and x.vector and not x.transcendental and made & x.read:
                need = max(need, 1)
            if p.m0 and x.memory and "lds" in x.text:
                need = max(need, 1)
            if p.vector and x.product and made & x.read:
                need = max(need, 2)
            if p.product:
                far = 11 if p.passes == 8 else 5
                if (x.vector and made & (x.read | x.written)) or (made & x.read and not x.product and not x.op.startswith("s_")):
                    need = far
                if x.product and made & (x.sources[0] | x.sources[1]):
                    need = far
                if x.vector and p.sources[2] - p.written & x.written:      # what the product starts from is read while it runs
                    need = max(need, 7 if p.passes == 8 else 1)
            if since < need:
                found.add((need, since, p.text, x.text))
            cost = stall(p) if p.product else p.states
            todo += [(q, since + cost, hidden | (p.written if len(hidden) < 64 else frozenset())) for q in p.before]
    return sorted(found)


LOAD = "buffer_load_dwordx4 v1, s[4:7], 0 offen lds"


@pytest.mark.parametrize("lines,count", [
    (["v_readfirstlane_b32 s6, v0", "s_mov_b32 m0, s9", "s_nop 0", LOAD], 1),
    (["v_readfirstlane_b32 s6, v0", "s_nop 2", "s_mov_b32 m0, s9", "s_nop 0", LOAD], 0),
    (["s_mul_i32 s6, s8, s9", "s_mov_b32 m0, s9", LOAD], 1),
    ([".LBB0_1:", "s_mov_b32 m0, s9", "s_nop 0", LOAD, "v_readfirstlane_b32 s7, v0", "s_cbranch_scc1 .LBB0_1", "s_endpgm"], 1),
    (["v_mfma_f32_32x32x16_bf16 v[8:23], v[0:3], v[4:7], 0", "s_cbranch_scc1 .LBB0_2", "s_nop 15", ".LBB0_2:", "v_exp_f32 v9, v1"], 1),
    (["v_mfma_f32_32x32x16_bf16 v[8:23], v[0:3], v[4:7], 0", "s_cbranch_scc1 .LBB0_2", "s_nop 15", ".LBB0_2:", "s_nop 9", "v_exp_f32 v9, v1"], 0),
    (["v_mfma_f32_32x32x16_bf16 v[8:23], v[0:3], v[4:7], v[24:39]", "s_nop 5", "v_mov_b32 v30, 0"], 1),
    (["v_exp_f32 v9, v1", "v_mul_f32 v2, v9, v9"], 1),
    (["v_exp_f32 v9, v1", "s_nop 0", "v_mul_f32 v2, v9, v9"], 0),
    (["v_mov_b32 v1, 0", "s_nop 0", "v_mfma_f32_32x32x16_bf16 v[8:23], v[0:3], v[4:7], v[8:23]"], 1)])
def test_the_check_follows_the_control_flow(lines, count):
    assert len(hazards(lines)) == count


@functools.lru_cache(maxsize=None)
def assembly(src, *defines):
    try:
        hipcc = B._hipcc()
    except RuntimeError:
        pytest.skip("hipcc not found")
    out = subprocess.run([hipcc, "-S", "--cuda-device-only", os.path.join(B.CSRC, src), "-o", "-"] + B.COMMON + B.DEVICE +
                         B.PER_FILE.get(src, []) + list(defines), check=True, stdout=subprocess.PIPE, stderr=subprocess.DEVNULL, text=True)
    return out.stdout.splitlines()


@pytest.mark.parametrize("src", SOURCES + [f"lf_attn.hip -DLF_PROBE -DLF_PROBE_{tag.upper()}" for tag in B.PROBES])
def test_instructions_keep_their_distance_on_every_path(src):
    """In wait states: a load behind the vector instruction that wrote its resource 5, behind M0 1; a vector instruction behind one
    that wrote a scalar register it reads 2, behind an exponential 1; a product behind a vector instruction 2; what uses a product's
    result 11 (4 x 4 x 4: 5), what overwrites the registers that a product starts from 7."""
    found = hazards(assembly(*src.split()))
    for f in found[:10]:
        print(*f)
    assert not found
