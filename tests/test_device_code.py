"""What the compiler makes of kernels whose loops count their own loads, from the assembly of this source (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2602_04789_amd import build as B


@pytest.fixture(scope="module")
def kv_wide(tmp_path_factory):
    """Kernel name -> lines of lf_attn_bwd_wide.hip as built."""
    try:
        hipcc = B._hipcc()
    except RuntimeError:
        pytest.skip("hipcc not found")
    out = str(tmp_path_factory.mktemp("asm") / "kv_wide.s")
    src = "lf_attn_bwd_wide.hip"
    subprocess.run([hipcc, "-S", "--cuda-device-only", os.path.join(B.CSRC, src), "-o", out] + B.COMMON + B.DEVICE +
                   B.PER_FILE.get(src, []), check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    kernels, name = {}, None
    with open(out) as f:
        for line in f:
            if re.match(r"_Z\w+:", line):
                name = line.split(":")[0]
                kernels[name] = []
            elif line.startswith(".Lfunc_end"):
                name = None
            elif name:
                kernels[name].append(line.split(";")[0].strip())
    assert len(kernels) == 2     # blocks with one and with two pairs of wavefronts
    return kernels


def test_loops_wait_for_counted_loads_only(kv_wide):
    """The loops of the two roles (two windows of 32 matrix instructions): no register is reloaded in them and nothing but
    the two counted waits of the loading role waits for memory, so the tile loads of two half tiles stay in flight."""
    for name, code in kv_wide.items():
        labels = {m[1]: i for i, l in enumerate(code) for m in [re.match(r"(\.LBB\w+):", l)] if m}
        loops = []
        for i, l in enumerate(code):
            m = re.match(r"s_c?branch\w*\s+(\.LBB\w+)", l)
            if m and labels[m[1]] < i and sum("v_mfma" in x for x in code[labels[m[1]]: i]) == 64:
                loops.append(code[labels[m[1]]: i])
        assert len(loops) == 2, name
        for body in loops:
            loads = sum("buffer_load" in x for x in body)
            waits = [re.search(r"vmcnt\((\d+)\)", x)[1] for x in body if "vmcnt" in x]
            print(name, "loads", loads, "waits", waits)
            assert loads in (0, 36) and waits == (["18", "18"] if loads else [])
            assert not any("scratch_" in x or "global_" in x for x in body)


def test_tile_loads_stand_behind_products_with_their_m0(kv_wide):
    """In the loading role's loop M0 is written only with the first load of each group of four (a product between them) and with
    each load of row statistics, and no scalar load counts with the LDS reads that the loop's waits count."""
    for name, code in kv_wide.items():
        code = [x for x in code if x]
        labels = {m[1]: i for i, l in enumerate(code) for m in [re.match(r"(\.LBB\w+):", l)] if m}
        ends = [(labels[m[1]], i) for i, l in enumerate(code) for m in [re.match(r"s_c?branch\w*\s+(\.LBB\w+)", l)] if m and labels[m[1]] < i]
        bodies = [code[a:b] for a, b in ends if sum("v_mfma" in x for x in code[a:b]) == 64]
        body = next(b for b in bodies if any("buffer_load" in x for x in b))
        m0 = [i for i, x in enumerate(body) if re.match(r"s_\w+ m0,", x)]
        print(name, "M0 written", len(m0))
        assert len(m0) == 12 and all("buffer_load" in body[i + 2] and re.match("v_", body[i + 1]) for i in m0)
        assert not any("m0" in x for i, x in enumerate(body) if i not in m0)
        loads = [i for i, x in enumerate(body) if "buffer_load_dwordx4" in x]
        assert len(loads) == 32 and all("v_mfma" in body[i - 1] for i in loads)
        assert not any(re.match(r"s_(buffer_)?load", x) for b in bodies for x in b)


def test_output_rows_are_staged_behind_a_barrier(kv_wide):
    """Output rows go through LDS where loaded tiles were (the only 8-byte LDS stores): behind the last products stand a wait
    for all loads, then a barrier, then the first of them."""
    for name, code in kv_wide.items():
        store = next(i for i, l in enumerate(code) if l.startswith("ds_write_b64"))
        product = max(i for i, l in enumerate(code[:store]) if "v_mfma" in l)
        wait = next((i for i in range(product, store) if "vmcnt(0)" in code[i]), store)
        print(name, "product", product, "wait", wait, "store", store)
        assert any("s_barrier" in l for l in code[wait:store])


def test_the_dq_loop_counts_its_loads(tmp_path):
    """The loop of dQ with one wavefront per query block (a window of 48 matrix instructions): 16 tile loads, one wait for the
    sixteen before, no other wait for memory; no register is reloaded, no scalar load counts with the LDS reads, and M0 is
    written only with the first load of each group of four."""
    try:
        hipcc = B._hipcc()
    except RuntimeError:
        pytest.skip("hipcc not found")
    src, out = "lf_attn_bwd_q_wide.hip", str(tmp_path / "q_wide.s")
    subprocess.run([hipcc, "-S", "--cuda-device-only", os.path.join(B.CSRC, src), "-o", out] + B.COMMON + B.DEVICE +
                   B.PER_FILE.get(src, []), check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    with open(out) as f:
        code = [x for x in (line.split(";")[0].strip() for line in f) if x]
    labels = {m[1]: i for i, l in enumerate(code) for m in [re.match(r"(\.LBB\w+):", l)] if m}
    loops = []
    for i, l in enumerate(code):
        m = re.match(r"s_c?branch\w*\s+(\.LBB\w+)", l)
        if m and labels[m[1]] < i and sum("v_mfma" in x for x in code[labels[m[1]]: i]) == 48:
            loops.append(code[labels[m[1]]: i])
    body = max(loops, key=len)         # (the masking of short half tiles branches back into it)
    waits = [x for x in body if "vmcnt" in x]
    print(waits)
    assert waits == ["s_waitcnt vmcnt(16)"] and sum("buffer_load" in x for x in body) == 16
    assert not any(re.match(r"(scratch|global|flat|s_load|s_buffer)_", x) for x in body)
    m0 = [i for i, x in enumerate(body) if re.match(r"s_\w+ m0,", x)]
    assert len(m0) == 4 and all(sum("buffer_load" in x for x in body[i: i + 3]) == 1 and "v_mfma" in body[i + 1] for i in m0)
    assert not any("m0" in x for i, x in enumerate(body) if i not in m0)


def _registers(text):
    out = set()
    for m in re.finditer(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        first, last = (m[2], m[3]) if m[2] else (m[4], m[4])
        out |= {(m[1], i) for i in range(int(first), int(last) + 1)}
    return out


def _hazards(code):
    """Pairs of a matrix and a vector instruction that stand closer than the hardware allows, in the order of the listing.
    History entries: text, kind, registers written, wait states from its issue to that of the next instruction."""
    bad, seen = [], []
    for line in code:
        m = re.match(r"([sv]_\w+|ds_\w+|buffer_\w+|global_\w+)\s*(.*)", line)
        if not m:
            continue
        op, args = m[1], re.split(r",\s*(?![^\[]*\])", m[2])
        product = "mfma" in op
        vector = op.startswith("v_") and not product
        written = _registers(args[0]) if product or vector else set()
        if "swap" in op:
            written |= _registers(args[1])
        read = _registers(" ".join(args[1:] if product or vector else args))
        cost = int(args[0], 0) + 1 if op == "s_nop" else 1
        since = 0
        for text, kind, regs, c in reversed(seen):
            if since >= 11:
                break
            if product and kind == "vector" and since < 2 and regs & read:
                bad.append((since, text, line))
            need = written | read if vector else read if not product and not op.startswith("s_") else set()
            if regs & need and since < {"mfma": 11, "small": 5}.get(kind, 0):
                bad.append((since, text, line))
            since += c
        if product:            # issues when the product before it has left the unit: 8 passes of four cycles
            since = 0
            for _, kind, _, c in reversed(seen):
                since += c
                if kind in ("mfma", "small"):
                    cost = max(1, (8 if kind == "mfma" else 2) - since)
                    break
        kind = ("small" if "4x4x4" in op else "mfma") if product else "vector" if vector else "other"
        seen = seen[-40:] + [(line, kind, written, cost)]
    return bad


def _assembly(src, tmp_path):
    try:
        hipcc = B._hipcc()
    except RuntimeError:
        pytest.skip("hipcc not found")
    out = str(tmp_path / "a.s")
    subprocess.run([hipcc, "-S", "--cuda-device-only", os.path.join(B.CSRC, src), "-o", out] + B.COMMON + B.DEVICE +
                   B.PER_FILE.get(src, []), check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    with open(out) as f:
        return [x for x in (line.split(";")[0].strip() for line in f) if x]


@pytest.mark.parametrize("src", ["lf_attn_wide.hip", "lf_attn_bwd_q_wide.hip", "lf_attn_bwd_wide.hip"])
def test_products_written_as_assembly_keep_their_distance(src, tmp_path):
    """What the compiler cannot see: a product needs two wait states behind a vector instruction that writes its source, a
    vector, LDS or memory instruction eleven behind the product whose result it uses (five behind a 4 x 4 x 4 one)."""
    assert _hazards(["v_mov_b32 v1, 0", "s_nop 0", "v_mfma_f32_32x32x16_bf16 v[8:23], v[0:3], v[4:7], v[8:23]"])
    assert _hazards(["v_mfma_f32_32x32x16_bf16 v[8:23], v[0:3], v[4:7], 0", "s_nop 8", "v_exp_f32 v9, v1"])
    assert not _hazards(["v_mov_b32 v1, 0", "s_nop 1", "v_mfma_f32_4x4x4_16b_bf16 v[8:11], v[0:1], v[4:5], 0", "s_nop 4",
                         "v_exp_f32 v9, v1"])
    assert _hazards(_assembly(src, tmp_path)) == []


def test_the_forward_loop_counts_its_loads(tmp_path):
    """The loop of the forward kernel with one wavefront per query block (two steps of 32 products of 32 x 32 x 16 and 8 sums): 16
    tile loads a step, two waits for the sixteen before, no register reloaded and no scalar load; M0 is written only with the
    first load of each group of four."""
    code = _assembly("lf_attn_wide.hip", tmp_path)
    labels = {m[1]: i for i, l in enumerate(code) for m in [re.match(r"(\.LBB\w+):", l)] if m}
    loops = []
    for i, l in enumerate(code):
        m = re.match(r"s_c?branch\w*\s+(\.LBB\w+)", l)
        if m and labels[m[1]] < i and sum("v_mfma_f32_32x32x16" in x for x in code[labels[m[1]]: i]) == 64:
            loops.append(code[labels[m[1]]: i])
    body = max(loops, key=len)
    waits = [x for x in body if "vmcnt" in x]
    print(waits)
    assert waits == ["s_waitcnt vmcnt(16)"] * 4 and sum("buffer_load" in x for x in body) == 32
    assert sum("v_mfma_f32_4x4x4" in x for x in body) == 16
    assert not any(re.match(r"(scratch|global|flat|s_load|s_buffer)_", x) for x in body)
    m0 = [i for i, x in enumerate(body) if re.match(r"s_\w+ m0,", x)]
    assert len(m0) == 8 and all(sum("buffer_load" in x for x in body[i: i + 3]) == 1 and "v_mfma" in body[i + 1] for i in m0)
    assert not any("m0" in x for i, x in enumerate(body) if i not in m0)
