"""The generated code of the kernels that live on loads in flight, the few-row GEMMs and decode attention (no GPU): nothing goes through
scratch memory, and their main loops never wait for all the loads they have under way.  The other attention kernels and the float q|k|v
product: nothing through scratch memory."""
import os
import re
import subprocess

import pytest

from paper_2603_13289_amd import build
from tests.test_gemm_code import _blocks


def _kernels(tmp_path, source, name):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path / "kernels.s")
    subprocess.run([build.HIPCC, *build.FLAGS, "--offload-device-only", "-S", os.path.join(build.CSRC, source), "-o", out],
                   check=True, capture_output=True)
    text = open(out).read()
    found = {m[1]: m[0].splitlines()[1:] for m in re.finditer(rf"^(_Z\w*{name}\w*):[^\n]*\n(.*?)^\.Lfunc_end", text, re.M | re.S)}
    scratch = {m[1]: int(m[2]) for m in re.finditer(
        r"\.amdhsa_kernel (\S+)\n(?:.*\n)*?\s*\.amdhsa_private_segment_fixed_size (\d+)", text)}
    return {k: (v, scratch[k]) for k, v in found.items()}


def _main_loops(lines):
    """Per loop that loads and multiplies: how many loads each wait in a multiplying block leaves in flight.  (Blocks without products may
    wait for the load of a block-table entry.)  Ranges of several blocks count where no such loop is a single block."""
    blocks = _blocks(lines)
    at = {label: i for i, (label, _) in enumerate(blocks) if label}
    spans = {(at[args], i) for i, (_, block) in enumerate(blocks) for op, args, _ in block
             if op.startswith(("s_cbranch", "s_branch")) and at.get(args, len(blocks)) <= i}
    loops = {}
    for first, last in spans:
        body = [block for _, block in blocks[first:last + 1]]
        products = [block for block in body if any("mfma" in op for op, _, _ in block)]
        if products and any(op.startswith("global_load") for block in body for op, _, _ in block):
            loops[first, last] = [int(n) for block in products for op, args, _ in block if op == "s_waitcnt"
                                  for n in re.findall(r"vmcnt\((\d+)\)", args)]
    return [w for span, w in loops.items() if span[0] == span[1]] or list(loops.values())


@pytest.mark.parametrize("source,name,count,loops", [("gemm_skinny.hip", "gemm_skinny_kernel", 14, 1),
                                                     ("gemm_skinny.hip", "gemm_wide_few_rows_kernel", 4, 1),
                                                     ("attention_mfma.hip", "attn_decode_kernel", 2, 2)])
def test_loads_stay_in_flight(tmp_path, source, name, count, loops):
    kernels = _kernels(tmp_path, source, name)
    assert len(kernels) == count
    for k, (lines, scratch) in kernels.items():
        assert scratch == 0 and not [l for l in lines if re.match(r"\s+scratch_", l)], k
        found = _main_loops(lines)
        assert len(found) >= loops, k
        assert all(waits and min(waits) > 0 for waits in found), (k, found)


@pytest.mark.parametrize("source,name,count", [("gemm_skinny.hip", "gemm_few_rows_parts_kernel", 4), ("attention_mfma.hip", "attn_mfma_kernel", 8),
                                               ("attention_mfma.hip", "attn_merge_kernel", 2), ("attention_f32.hip", "attn_f32_kernel", 4),
                                               ("gemm_f32.hip", "gemm_f32_rope_kernel", 2)])
def test_no_scratch(tmp_path, source, name, count):
    kernels = _kernels(tmp_path, source, name)
    assert len(kernels) == count
    assert all(scratch == 0 for _, scratch in kernels.values())
