"""What a short call pays for: work that only longer calls need must stand
behind a branch (CPU: the compiled kernels; GPU: results at those sizes)."""
import os
import re

import pytest

from tests.test_kernel_fragments import CSRC, blocks_of
from tests.test_kernel_structure import asm_of


def _kernels(asm, name):
    found = sorted(set(re.findall(rf"^(_ZN4asym\S*{name}\S*):", asm, re.M)))
    assert found, name
    return found


@pytest.mark.parametrize("src,name", [("attn_decode.hip", "attn_decode_merge"), ("mla_decode.hip", "mla_decode_merge")])
def test_merge_loads_only_the_splits_there_are(tmp_path, src, name):
    """A wave's first eight splits are loaded one by one, each behind a branch,
    so a row of one split costs one split's loads; whole batches stand in the
    loop over further splits alone."""
    asm = asm_of(src, tmp_path)
    for k in _kernels(asm, name):
        loads = [sum(i.startswith("global_load") for i, _ in b["insts"]) for b in blocks_of(asm, k)]
        assert sum(n > 4 for n in loads) <= 1, (k, loads)
        assert sum(n in (2, 3) for n in loads) >= 8, (k, loads)


def test_small_m_ring_loads_only_the_stages_there_are(tmp_path):
    """The ring is filled in one run only where K fills it; a shorter K loads its
    stages in a loop, and the last stages of any K load nothing."""
    asm = asm_of("gemm_skinny.hip", tmp_path)
    for k in _kernels(asm, "gemm_bf16_small_mI"):
        lps = 4 if "ILi4E" in k else 3
        loads, mfmas = [], []
        for b in blocks_of(asm, k):
            loads.append(sum(bool(re.match(r"buffer_load.*\blds$", i)) for i, _ in b["insts"]))
            mfmas.append(sum(i.startswith("v_mfma") for i, _ in b["insts"]))
        assert sum(n > 2 * lps for n in loads) == 1, (k, loads)
        assert any(n == lps and not m for n, m in zip(loads, mfmas)), (k, loads)
        assert loads[mfmas.index(max(mfmas))] == 0, (k, loads, mfmas)


def test_the_ring_depth_counts_the_streams_cus():
    """The deep ring takes a whole CU: it is for launches of one workgroup per CU of the set they run on."""
    capi, skinny = (open(os.path.join(CSRC, f)).read() for f in ("capi.cpp", "gemm_skinny.hip"))
    assert capi.count("  SmallMLaunch sm;\n") == 2 == capi.count("sm.set_cus = P.total;")
    assert "const bool deep = grid <= g.set_cus;" in skinny
