"""The generated code of the q|k|v product with rotary in its epilogue keeps the same promise as the plain pipelined GEMM (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2603_13289_amd import build
from tests.test_gemm_code import _blocks, _touched_in_flight


def test_no_fragment_is_touched_early_or_spilled(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path / "gemm.s")
    subprocess.run([build.HIPCC, *build.FLAGS, "--offload-device-only", "-S", os.path.join(build.CSRC, "gemm_mfma.hip"), "-o", out],
                   check=True, capture_output=True)
    text = open(out).read()
    found = {m[1]: m[0].splitlines()[1:] for m in
             re.finditer(r"^(_Z\w*gemm_qkv_rope_kernel\w*TilePipe\w*):[^\n]*\n(.*?)^\s*s_endpgm.*?^\.Lfunc_end", text, re.M | re.S)}
    assert len(found) == 8           # eight tile types
    for name, lines in found.items():
        blocks = _blocks(lines)
        assert sum(in_asm and op == "ds_read_b128" for _, b in blocks for op, _, in_asm in b) >= 32, name
        assert not _touched_in_flight(blocks), name
        assert not [l for l in lines if re.match(r"\s+scratch_", l)], name
        assert {m[1] for l in lines if (m := re.match(r"\s+(global_store_\w+)", l))} == {"global_store_dwordx2", "global_store_dwordx4"}, name
