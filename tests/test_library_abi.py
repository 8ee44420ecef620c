"""No-GPU checks of the boundary: the library loads and exports what include/lrqmm.h declares."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    with open(os.path.join(ROOT, "include", "lrqmm.h")) as f:
        text = f.read()
    return sorted(set(re.findall(r"LRQMM_API[^;(]*?\b(lrqmm_\w+)\s*\(", text)))


def test_header_declares_the_three_named_calls():
    names = _declared()
    for n in ("lrqmm_quantize", "lrqmm_rsvd", "lrqmm_gemm", "lrqmm_matmul", "lrqmm_fill_sketch",
              "lrqmm_workspace_bytes", "lrqmm_status_string", "lrqmm_profile_enable", "lrqmm_profile_read"):
        assert n in names


def test_library_exports_every_declared_symbol():
    import paper_2409_18772_amd as L
    if not os.path.exists(L.lib_path()):
        pytest.skip("library not built (run __graft_entry__.build())")
    lib = ctypes.CDLL(L.lib_path())
    for n in _declared():
        assert hasattr(lib, n), n
    assert set(_declared()) == set(L.binding.EXPORTS)


def test_host_side_validation_without_a_gpu():
    import paper_2409_18772_amd as L
    if not os.path.exists(L.lib_path()):
        pytest.skip("library not built")
    lib = L.load_library()
    assert L.lrqmm_status_string(0) == "ok"
    assert "workspace" in L.lrqmm_status_string(-3)
    assert L.lrqmm_workspace_bytes(-1, 4, 4, 0, 0) == 0
    assert L.lrqmm_workspace_bytes(64, 64, 64, 70, 20) == 0
    small, big = L.lrqmm_workspace_bytes(256, 256, 256, 8, 0), L.lrqmm_workspace_bytes(4096, 4096, 4096, 32, 8)
    assert 0 < small < big
    assert big % 1 == 0 and big >= 2 * 4096 * 4096
    # argument checks return before anything touches a device
    assert lib.lrqmm_quantize(None, 4, 4, 0, 1, 0, None, None, None) == -2
    assert lib.lrqmm_quantize(None, 4, 4, 5, 8, 0, None, None, None) == -1
    assert lib.lrqmm_quantize(None, 4, 4, 0, 8, 0, None, None, None) == -1
    assert lib.lrqmm_rsvd(None, None, 8, 8, 0, 8, 0, 0, 0, 0, 0, None, None, None, None, None, 0, None) == -1
    assert lib.lrqmm_rsvd(None, None, 8, 8, 0, 8, 0, 9, 0, 0, 0, None, None, None, None, None, 0, None) == -1
    assert lib.lrqmm_rsvd(None, None, 200, 200, 0, 8, 0, 81, 0, 0, 0, None, None, None, None, None, 0, None) == -2
    assert lib.lrqmm_gemm(4, 4, 1 << 20, 8, 0, *([None] * 12), None, 0, None) == -2
    assert lib.lrqmm_matmul(4, 4, 4, 8, 5, 0, 0, 0, 0, None, None, None, None, 0, None) == -1
    assert lib.lrqmm_fill_sketch(1, -1, 4, 4, None, None) == -1
    # strides below the row length, unknown scale granularity
    assert lib.lrqmm_quantize_ex(None, 3, 4, 4, 0, 8, 0, 0, None, None, None) == -1
    assert lib.lrqmm_quantize_ex(None, 4, 4, 4, 0, 8, 0, 7, None, None, None) == -1
    assert lib.lrqmm_rsvd_ex(None, 7, None, 8, 8, 0, 8, 0, 2, 0, 0, 0, None, 0, None, None, None, None, 0, None) == -1
    assert lib.lrqmm_rsvd_ex(None, 8, None, 8, 8, 0, 8, 0, 2, 0, 0, 0, None, 3, None, None, None, None, 0, None) == -1     # unknown precision
    assert lib.lrqmm_gemm_ex(4, 4, 4, 8, 0, *([None] * 10), 1.0, 0.0, None, 3, None, None, 0, None) == -1
    assert lib.lrqmm_matmul_ex(4, 4, 4, 8, 0, 0, 0, 0, 0, 0, 0, None, 3, None, 4, 1.0, 0.0, None, 4, None, 0, None) == -1
    assert lib.lrqmm_matmul_ex(4, 4, 4, 8, 0, 0, 0, 0, 0, 3, 0, None, 4, None, 4, 1.0, 0.0, None, 4, None, 0, None) == -1
    assert lib.lrqmm_matmul_ex(4, 4, 4, 8, 0, 0, 0, 0, 0, 0, 5, None, 4, None, 4, 1.0, 0.0, None, 4, None, 0, None) == -1     # unknown precision


@pytest.mark.parametrize("M,N,K", [(0, 96, 80), (64, 0, 80), (64, 96, 0), (0, 0, 0)])
def test_workspace_of_an_empty_problem(M, N, K):
    """An extent of zero with rank > 0: the size query returns, an empty product is accepted and a rank above K refused
    (in a child process: an integer division by zero would end the interpreter)."""
    import subprocess
    import sys
    import paper_2409_18772_amd as L
    if not os.path.exists(L.lib_path()):
        pytest.skip("library not built")
    code = (f"import paper_2409_18772_amd as L; lib = L.load_library();"
            f"print(L.lrqmm_workspace_bytes({M}, {N}, {K}, 8, 4),"
            f"lib.lrqmm_gemm_static({M}, {N}, {K}, 8, 8, *([None] * 10), 1.0, 0.0, None, {N}, None, None))")
    p = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stderr
    nbytes, status = (int(x) for x in p.stdout.split())
    assert nbytes > 0
    assert status in ((0,) if M == 0 or N == 0 else (-1, -4))       # (-4: no GPU to look the static scratch up on)


def test_workspace_counts_only_what_can_run():
    """The sums of the kernel that reads a tall A once lie over the passes' partial results, and factors in the order of steps are
    counted up to the longest that take that order."""
    import paper_2409_18772_amd as L
    if not os.path.exists(L.lib_path()):
        pytest.skip("library not built")
    size = L.lrqmm_workspace_bytes
    # A sketch of 80 columns over 4096 values a row never reads A once: no step where tall operands begin, 25001 rows; a row more costs its
    # codes and factors, and up to 64 rows of partial results (the kernel's sums would be 19 million bytes).
    for rows in (20000, 25000, 32768):
        assert size(rows + 1, 64, 4096, 64, 16) - size(rows, 64, 4096, 64, 16) < 1_000_000
    # Without either the two calls take 86 and 592 million bytes; a row of 16 columns in the order of steps takes 96, the
    # kernel's sums are 19 million of which 8 lie over partial results; for 80 columns 256 Gram partials an operand in place of 64 and
    # 8192 rows in the order of steps.
    assert size(100352, 64, 576, 8, 0) < 86e6 + 96 * 100352 + 12e6
    assert size(100352, 64, 4096, 64, 16) < 592e6 + 96 * 100352 + 2 * (192 * 80 * 80 * 8 + 8192 * 480)


def test_workspace_of_a_larger_problem_serves_a_smaller_one():
    """The size does not fall when an extent, the rank or the oversampling grows.  Extents around the limits of the launch
    plans (512 blocks of 64 rows, 1024 rows, 256 x 256 tiles) and pairs that the plans treat very differently."""
    import random
    import paper_2409_18772_amd as L
    if not os.path.exists(L.lib_path()):
        pytest.skip("library not built")
    size = L.lrqmm_workspace_bytes
    assert size(288, 2053, 1604, 16, 0) <= size(359, 2053, 1604, 16, 0)
    assert size(224, 691, 3550, 16, 0) <= size(228, 691, 3550, 16, 0)
    assert size(4096, 4096, 4096, 32, 8) <= size(4100, 4096, 4096, 32, 8)
    rng = random.Random(5)
    edges = [64, 255, 256, 511, 512, 1023, 1024, 1025, 2048, 4096, 4097, 8192, 8193, 32704, 32705, 32768, 65536]

    def extent():
        return rng.choice(edges) if rng.random() < 0.3 else int(2 ** rng.uniform(5, 17))
    for _ in range(20000):
        big = [extent() for _ in range(3)] + [rng.randint(1, 64), rng.choice([0, 4, 8, 16])]
        small = list(big)
        for i in rng.sample(range(5), rng.choice([1, 1, 2, 5])):
            low = 1 if i < 4 else 0
            small[i] = rng.randint(max(low, big[i] - 40), big[i]) if rng.random() < 0.5 else rng.randint(low, big[i])
        if rng.random() < 0.1 and small[3] > 0:
            small[3] = 0
        assert size(*small) <= size(*big), (small, big)


def test_missing_library_fails_loudly(monkeypatch, tmp_path):
    import paper_2409_18772_amd.binding as b
    monkeypatch.setattr(b, "_LIB", None)
    monkeypatch.setattr(b, "_HERE", str(tmp_path))
    with pytest.raises(ImportError):
        b.load_library()
