"""GEMM tiles computed in parts (the deep-ring kernel).

CPU: the compiled kernels' accumulators are neither read before the MFMA fence
nor written too late before an MFMA, and each claim is published in its own
loop.  GPU: every part shape at the edges of its range (K of one stage, of
fewer and more stages than ring slots, odd and even stage counts, ragged K;
rows and columns that leave parts empty or end inside one), element by element
against the oracle and, on integers, bit for bit.
"""
import os
import subprocess

import numpy as np
import pytest
import torch

import oracle
import paper_2609_24270_amd as asym
from paper_2609_24270_amd import workloads
from tests.checks import assert_gemm_close
from tests.test_kernel_fragments import (CSRC, ROOT, _split, _vregs, blocks_of, inflight_violations,
                                         write_to_mfma_violations)
from tests.test_kernel_structure import annotate_loops, asm_of, claims_published_in_their_loop, function_body

# FM, FN, ring slots, direct loads into LDS
PARTS = [(4, 6, 4, 1), (4, 4, 4, 1), (4, 3, 4, 1), (4, 2, 6, 1), (2, 2, 6, 1), (4, 4, 3, 0), (4, 2, 3, 0), (2, 2, 3, 0)]


@pytest.fixture(scope="module")
def part_asm(tmp_path_factory):
    return asm_of("gemm.hip", tmp_path_factory.mktemp("asm"))


@pytest.mark.parametrize("fm,fn,ns,dma", PARTS)
def test_part_kernel_hazards_and_claims(part_asm, fm, fn, ns, dma):
    name = f"gemm_bf16_partsILi{fm}ELi{fn}ELi{ns}ELb{dma}ELb0E"
    kernel = f"_ZN4asym12_GLOBAL__N_115{name}EEvNS0_6ParamsE"
    v = inflight_violations(part_asm, kernel)
    assert not v, f"{len(v)} accumulator accesses before the MFMA fence, e.g. {v[:4]}"
    v = write_to_mfma_violations(part_asm, kernel)
    assert not v, f"{len(v)} asm MFMAs too soon after an accumulator write, e.g. {v[:3]}"
    v = operand_violations(part_asm, kernel)
    assert not v, v[:4]
    insts = annotate_loops(function_body(part_asm, name))
    assert claims_published_in_their_loop(
        insts, r"^global_atomic_add v\d+, v\d+, v\d+, s\[\d+:\d+\]( offset:\d+)? sc0") >= 1


def operand_violations(asm, kernel, min_states=2):
    """Inline-asm MFMAs within `min_states` wait states after a compiler-placed
    vector instruction of the same block that writes one of their A or B
    operands (the compiler does not know the asm to be an MFMA)."""
    out = []
    for b in blocks_of(asm, kernel):
        recent = {}  # VGPR -> wait states since a vector instruction wrote it
        for inst, is_asm in b["insts"]:
            mn, writes, _ = _split(inst)
            if is_asm and mn.startswith("v_mfma"):
                a, bb = (x.strip() for x in inst.split(None, 1)[1].split("],", 3)[1:3])
                hit = [r for r in _vregs(a + "]") | _vregs(bb + "]") if recent.get(r, 99) < min_states]
                if hit:
                    out.append((b["label"], inst, hit))
            step = int(inst.split()[1]) + 1 if mn == "s_nop" else 1
            recent = {r: n + step for r, n in recent.items() if n + step < min_states}
            if not is_asm and mn.startswith("v_") and not mn.startswith("v_mfma"):
                recent.update({r: 0 for r in writes})
    return out


def test_operand_rule_sees_a_planted_write():
    bad = "k:\n; %bb.0:\n\tv_mov_b32_e32 v5, v9\n\t;;#ASMSTART\n\tv_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]\n\t;;#ASMEND\n.Lfunc_end0:\n"
    assert operand_violations(bad, "k")
    assert not operand_violations(bad.replace("\t;;#ASMSTART", "\ts_nop 7\n\t;;#ASMSTART", 1), "k")


@pytest.mark.parametrize("form", [1, 2, 3, 4])  # 3, 4: non-temporal rows
def test_latent_attention_workgroup_forms_hazards(tmp_path, form):
    asm = _asm_vgpr_form("mla_decode.hip", tmp_path)
    kernel = f"_ZN4asym12_GLOBAL__N_119mla_decode_split_wgILi{form}EEEvNS0_9MlaParamsE"
    assert not inflight_violations(asm, kernel)
    assert not write_to_mfma_violations(asm, kernel)
    v = operand_violations(asm, kernel)
    assert not v, v[:4]


def _asm_vgpr_form(src, tmp_path):
    out = tmp_path / "k.s"
    cmd = ["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-I", os.path.join(ROOT, "include"),
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-mllvm", "-amdgpu-mfma-vgpr-form=1",
           "--cuda-device-only", "-S", os.path.join(CSRC, src), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out.read_text()


def bits(t):
    return t.detach().cpu().contiguous().view(torch.int16).numpy().view(np.uint16)


# On 256 CUs: 64 x 64 parts up to 64 tiles of 128 x 128, 128 x 64 up to 128,
# 128 x 96 while those number at most 256, else 128 x 128; 128 x 192 where half
# of the 256-row tiles' count fits.  More than 256 rows (fewer run on the
# small-M kernel).
SHAPES = [
    (257, 72, 8), (257, 200, 64), (300, 500, 72), (513, 130, 448), (321, 1000, 456),        # 64 x 64
    (1100, 1100, 8), (1100, 1100, 328), (513, 2500, 520),                                    # 128 x 64
    (1100, 2500, 64), (1030, 2304, 200), (700, 3700, 456),                                   # 128 x 96
    (2048, 2048, 72), (2000, 2040, 264),                                                     # 128 x 128
    (2100, 2500, 8), (2304, 2048, 200), (2500, 2300, 328),                                   # 128 x 192
]
# operands on 2-byte boundaries: (M, N, K, elements each row is longer than K)
ODD = [(1, 1, 1, 0), (17, 33, 7, 2), (300, 130, 9, 0), (70, 257, 63, 1), (300, 300, 64, 3), (200, 700, 255, 0),
       (1100, 1101, 256, 1), (65, 1000, 257, 0), (1111, 1111, 263, 0), (2050, 1999, 319, 0), (2050, 1999, 321, 5),
       (2500, 2301, 384, 7), (129, 515, 447, 0), (1000, 3001, 449, 0), (333, 77, 1003, 0)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_parts_elementwise_and_bitwise(M, N, K):
    dev = torch.device("cuda:0")
    for dist in ("uniform", "int"):
        A, B = workloads.make_inputs(workloads.make_problem(M, N, K, seed=M + N + K, dist=dist))
        R, Co = oracle.gemm_bf16(bits(A), bits(B), "nk")
        Ad, Bd = A.to(dev), B.to(dev)
        ref = None
        for kw in ({}, {"mapping": "oblivious_rowmajor"}, {"xcd_mask": 0x0D}):  # static, whole order, claims
            C = torch.full((M, N + 12), 3.0, dtype=torch.bfloat16, device=dev)
            asym.gemm(Ad, Bd, C[:, :N], **kw)
            torch.cuda.synchronize()
            assert torch.all(C[:, N:].cpu() == 3.0), kw  # nothing past N
            got = bits(C[:, :N])
            if ref is None:
                ref = got
                if dist == "int":
                    assert np.array_equal(got, Co)
                else:
                    assert assert_gemm_close(got, R, what=f"{M}x{N}x{K}") < 5e-3
            assert np.array_equal(got, ref), kw


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,pad", ODD)
def test_unaligned_operands(M, N, K, pad):
    """Rows of any length from any 2-byte boundary, with NaNs before the first
    element, behind each row and behind the last one: none of them is used,
    nothing beside C is written, and every mapping gives the oracle's bits on
    integers."""
    dev = torch.device("cuda:0")

    def placed(x, lead):
        r, k = x.shape
        buf = torch.full((lead + r * (k + pad) + 8,), float("nan"), dtype=torch.bfloat16, device=dev)
        v = buf[lead:lead + r * (k + pad)].view(r, k + pad)
        v[:, :k] = x.to(dev)
        return v[:, :k]

    for dist in ("uniform", "int"):
        A, B = workloads.make_inputs(workloads.make_problem(M, N, K, seed=M + N + K, dist=dist))
        R, Co = oracle.gemm_bf16(bits(A), bits(B), "nk")
        for lead, kw in ((1, {}), (3, {"mapping": "oblivious_grouped"}), (5, {"xcd_mask": 0x81})):
            Ad, Bd = placed(A, lead), placed(B, 8 - lead)
            cb = torch.full((lead + M * (N + pad) + 8,), 3.0, dtype=torch.bfloat16, device=dev)
            C = cb[lead:lead + M * (N + pad)].view(M, N + pad)[:, :N]
            assert asym.gemm_plan(Ad, Bd, C, **kw)["vector_path"] == 0
            asym.gemm(Ad, Bd, C, **kw)
            torch.cuda.synchronize()
            got = bits(C)
            C.fill_(3.0)
            assert torch.all(cb.cpu() == 3.0), kw
            if dist == "int":
                assert np.array_equal(got, Co), kw
            else:
                assert assert_gemm_close(got, R, what=f"{M}x{N}x{K} {kw}") < 5e-3


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(700, 301, 72), (2048, 2047, 200), (2300, 2303, 136), (2600, 4003, 200)])
def test_aligned_operands_into_unaligned_c(M, N, K):
    """A and B on the vector path, rows of C from any 2-byte boundary."""
    dev = torch.device("cuda:0")
    A, B = workloads.make_inputs(workloads.make_problem(M, N, K, seed=M, dist="int"))
    _, Co = oracle.gemm_bf16(bits(A), bits(B), "nk")
    C = torch.full((M, N + 2), 3.0, dtype=torch.bfloat16, device=dev)
    assert asym.gemm_plan(A.to(dev), B.to(dev), C[:, 1:N + 1])["vector_path"] == 1
    asym.gemm(A.to(dev), B.to(dev), C[:, 1:N + 1])
    torch.cuda.synchronize()
    assert np.array_equal(bits(C[:, 1:N + 1]), Co)
    assert torch.all(C[:, 0].cpu() == 3.0) and torch.all(C[:, N + 1].cpu() == 3.0)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(300, 520, 264), (512, 6144, 512), (1024, 6144, 512), (300, 521, 263)])
def test_part_trace_records(M, N, K):
    """Records of a product computed in parts: each tile counted once, `worked` and `first_tile` together, and the
    claiming form's first part begins behind its rank ticket and claim: two atomics' round trips (1.6 us; the
    workgroup's setup is the same in both forms).  1024 x 6144 on four XCDs is whole tiles, some workers without one."""
    dev = torch.device("cuda:0")
    topo = asym.probe_topology(0, asym.PROBE_IDENTITY)
    A, B = (x.to(dev) for x in workloads.make_inputs(workloads.make_problem(M, N, K, seed=41)))
    prev = asym.set_small_m(False)
    try:
        ref = asym.gemm(A, B, topo=topo)
    finally:
        asym.set_small_m(prev)
    khz = asym.device_query(0)["wall_clock_khz"]
    leads = []
    for xcd_mask in (0, 0x0F):
        C = torch.zeros_like(ref)
        t = asym.gemm_trace(A, B, C, topo=topo, xcd_mask=xcd_mask, launches=2)[1]  # (the second: the kernel is loaded)
        assert torch.equal(C, ref)
        assert t["plan"]["claims"] == (xcd_mask != 0) and len(t["tiles"]) == t["plan"]["grid"]
        assert int(t["tiles"].sum()) == t["plan"]["tiles_m"] * t["plan"]["tiles_n"]
        worked = t["worked"] == 1
        assert np.array_equal(worked, t["first_tile"] != 0) and worked.any()
        assert (t["tiles"][~worked] == 0).all()
        first = t["first_tile"][worked]
        assert (first >= t["start"][worked]).all() and (first <= t["end"][worked]).all()
        leads.append(np.median((first - t["start"][worked]).astype(np.float64)) / khz * 1e3)
    print(f"{M}x{N}x{K}: first part {leads[0]:.2f} us after the start, claimed {leads[1]:.2f}")
    assert leads[1] >= leads[0] + 0.5
