"""The generated code of the pipelined GEMM keeps the promise its inline-assembly LDS reads rest on (no GPU).

The compiler believes that such a read has delivered its registers at once.  So no instruction may read or write them
before a wait for LDS reads, on any path, and nothing may be spilled."""
import os
import re
import subprocess

import pytest

from paper_2603_13289_amd import build


def _registers(text):
    out = set()
    for lo, hi, one in re.findall(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b", text):
        out |= set(range(int(lo), int(hi) + 1)) if lo else {int(one)}
    return out


def _blocks(lines):
    """[(label or None, [(instruction, operands, inside inline assembly)])] in program order."""
    blocks, in_asm = [(None, [])], False
    for line in lines:
        if ";;#ASM" in line:
            in_asm = "START" in line
        elif re.match(r"\.LBB\w+:", line):
            blocks.append((line.split(":")[0], []))
        else:
            m = re.match(r"\s+([a-z][a-z_0-9]+)\s*([^;]*)", line)
            if m:
                blocks[-1][1].append((m[1], m[2].strip(), in_asm))
                if m[1].startswith(("s_cbranch", "s_branch", "s_endpgm")):
                    blocks.append((None, []))
    return blocks


def _touched_in_flight(blocks):
    at = {label: i for i, (label, _) in enumerate(blocks) if label}
    seen, work, bad = {0: frozenset()}, [0], set()
    while work:
        i = work.pop()
        flying, successors, falls = set(seen[i]), [], True
        for op, args, in_asm in blocks[i][1]:
            if op == "s_waitcnt":
                flying = set() if "lgkmcnt(0)" in args else flying
                continue
            if _registers(args) & flying:
                bad.add(f"{op} {args}")
            if in_asm and op == "ds_read_b128":
                flying |= _registers(args.split(",")[0])
            if op.startswith(("s_cbranch", "s_branch")):
                successors.append(at[args])
            falls = falls and op not in ("s_branch", "s_endpgm")
        for j in successors + ([i + 1] if falls and i + 1 < len(blocks) else []):
            new = frozenset(flying) | seen.get(j, frozenset())
            if j not in seen or new != seen[j]:
                seen[j] = new
                work.append(j)
    return bad


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("asm") / "gemm.s")
    subprocess.run([build.HIPCC, *build.FLAGS, "--offload-device-only", "-S",
                    os.path.join(build.CSRC, "gemm_mfma.hip"), "-o", out], check=True, capture_output=True)
    text = open(out).read()
    found = {}
    for m in re.finditer(r"^(_Z\w*gemm_mfma_dl_kernel\w*TilePipe\w*):[^\n]*\n(.*?)^\s*s_endpgm.*?^\.Lfunc_end", text, re.M | re.S):
        found[m[1]] = m[0].splitlines()[1:]
    assert len(found) == 14          # eight tile types, two of them without the gate/up form
    return found


def test_nothing_touches_a_fragment_before_the_wait(kernels):
    for name, lines in kernels.items():
        blocks = _blocks(lines)
        reads = sum(in_asm and op == "ds_read_b128" for _, b in blocks for op, _, in_asm in b)
        assert reads >= 32, name
        assert not _touched_in_flight(blocks), name


def test_nothing_is_spilled(kernels):
    for name, lines in kernels.items():
        assert not [l for l in lines if re.match(r"\s+scratch_", l)], name


def test_gate_up_outputs_are_stored_eight_bytes_at_a_time(kernels):
    """One by one at the ragged end of a row, else four bf16 outputs with one store; K parts 16 bytes at a time."""
    gate_up = {name: lines for name, lines in kernels.items() if re.search(r"EELb1ELb[01]E", name)}
    assert len(gate_up) == 6
    for name, lines in gate_up.items():
        stores = [m[1] for l in lines if (m := re.match(r"\s+(global_store_\w+)", l))]
        assert set(stores) == {"global_store_short", "global_store_dwordx2", "global_store_dwordx4"}, name
        assert stores.count("global_store_short") == 4 * stores.count("global_store_dwordx2"), name
