"""The rules for non-temporal loads (CPU: the host functions themselves)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_24270_amd", "csrc")
MIB = 1 << 20


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    """rule(expression) -> the value of a C++ expression over read_policy.h."""
    def run(*exprs):
        d = tmp_path_factory.mktemp("policy")
        src = d / "p.cpp"
        src.write_text('#include <cstdio>\n#include "read_policy.h"\nusing namespace asym;\nint main() {\n' +
                       "".join(f'std::printf("%lld\\n", (long long)({e}));\n' for e in exprs) + "}\n")
        r = subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(d / "p")],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        return [int(x) for x in subprocess.run([str(d / "p")], capture_output=True, text=True).stdout.split()]
    return run


def test_attention_reads_what_the_caches_keep_with_ordinary_loads(rule):
    # B=1 x 32768 and B=4 x 8192 tokens of 8 heads are 128 MiB, the sizes of placed pages
    sizes = [33 * MIB, 128 * MIB, 200 * MIB, 256 * MIB - 1, 256 * MIB, 500 * MIB, 8192 * MIB]
    assert rule(*(f"attn_streams_kv({s}ll)" for s in sizes)) == [0, 0, 0, 0, 1, 1, 1]


def test_small_cu_sets_read_with_ordinary_loads(rule):
    assert rule(*(f"attn_set_streams({n}, 256)" for n in (64, 128, 224, 239, 240, 256))) == [0, 0, 0, 0, 1, 1]


def test_pages_that_requests_share_count_once(rule):
    # 64 requests x 8 heads x 4096 tokens over the pages of one of them: 16 MiB
    assert rule(f"paged_kv_bytes({1024 * MIB}ll, {8 * MIB}ll, false)", f"paged_kv_bytes({1024 * MIB}ll, {8 * MIB}ll, true)",
                f"paged_kv_bytes({1024 * MIB}ll, {2048 * MIB}ll, true)", f"paged_kv_bytes({100 * MIB}ll, {400 * MIB}ll, false)",
                f"attn_streams_kv(paged_kv_bytes({1024 * MIB}ll, {8 * MIB}ll, false))") == [
                    16 * MIB, 8 * MIB, 1024 * MIB, 100 * MIB, 0]


def test_pages_of_a_thin_second_round_are_not_streamed(rule):
    def thin(g, tasks, round=2048):
        return f"pages_thin_round({g}, {tasks}, {round})"
    # one round, a second one of 1/8 and less, of 1/4, of 5/8 and past it, two rounds, more of them
    assert rule(*(thin(1, t) for t in (2048, 2304, 2305, 2560, 3328, 3329, 4096, 4608))) == [0, 0, 1, 1, 1, 0, 0, 0]
    assert rule(thin(2, 2560), thin(4, 2560), thin(1, 1280, 1024), thin(1, 100)) == [1, 0, 1, 0]


def test_weights_stream_by_whole_lines_only(rule):
    def b(at, ldb, mib, steps=0):
        return f"small_m_streams_b((const void*){at}, {ldb}, {mib * MIB}ll, {steps})"
    assert rule(b(4096, 4096, 64), b(4096, 4096, 63), b(4096, 2048, 512)) == [1, 0, 1]
    # a pitch of half lines, a first row inside a line, k ranges that start inside one
    assert rule(b(4096, 2040, 125), b(4096, 4088, 512), b(4096 + 16, 4096, 112), b(4096 + 64, 4096, 112),
                b(4096, 4096, 112, 16), b(4096, 4096, 112, 15)) == [0, 0, 0, 0, 1, 0]


def test_a_fresh_copy_is_read_from_the_caches(rule):
    def b(mib, fresh):
        return f"small_m_streams_b((const void*)4096, 4096, {mib * MIB}ll, 0, {fresh})"
    assert rule(b(112, 0), b(112, 1), b(127, 1), b(128, 1)) == [1, 0, 0, 1]


def test_the_launch_asks_the_rules():
    capi = open(os.path.join(CSRC, "capi.cpp")).read()
    assert "a.once = attn_streams_kv(kv_bytes) && attn_set_streams(P.cs.total, P.cs.t->n_cus);" in capi
    assert "if (paged && pages_thin_round(Hq / Hkv, P.tasks, " in capi
    assert "kv_bytes = paged_kv_bytes(kv_bytes, a.pool_bytes, k == v)" in capi
    assert capi.count("small_m_streams_b(B, ldb, ") == 2 and capi.count("b_once = ") == 2
    # the [K][N] path says that its B is a copy of this call
    assert capi.count("ws->kn_buf, ldt, ASYM_B_NK, C, ldc, mapping, xcd_mask,\n                          stream, true)") == 1
    assert "range_steps, b_fresh)" in capi and "lda, ldb, ldc, mapping, b_fresh)" in capi
