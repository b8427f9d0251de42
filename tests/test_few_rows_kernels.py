"""The compiled kernels of a pass of few rows are those that a rule can reach, and what has no kernel is refused, on the CPU."""
import ctypes as C
import re
import subprocess
import pytest
from test_abi_cpu import lib  # noqa: F401

F32, BF16 = 0, 1
RESID, NORM_GEMM = "_ZN8sprinter17launch_gemm_residEiiPKvS1_iiPKfPfS4_iP12ihipStream_t", "_ZN8sprinter16launch_norm_gemmEiiiPKfS1_S1_S1_fPKNS_11EmbedSourceEPfPKvS7_iiS1_PviP12ihipStream_t"
WIDTHS = range(64, 8193, 64)


def _compiled(lib, kernel):
    from paper_2502_04557_amd import binding
    names = subprocess.run(["nm", "-C", binding.LIB_PATH], capture_output=True, text=True, check=True).stdout
    return {tuple(t.strip() for t in m.split(",")) for m in re.findall(r"sprinter::" + kernel + r"<([^<>]*)>\(", names)}


def _takes_norm(lib, dtype, d, rows):
    return bool(lib["_ZN8sprinter15gemm_takes_normEiii"](dtype, d, rows) & 0xFF)


def _resid_kernel(dtype, N, K, rows):
    """(type, S, RP, UG, MT): columns per workgroup 16 / S, rows per activation load, groups of k tiles in flight, operands of 16 rows."""
    S = 1 if N > 2048 else 4 if dtype == F32 and N <= 1024 and rows <= 4 else 2
    if rows > 16:
        return "unsigned short", S, 16, 8 if S == 1 else 4, 2
    RP = 4 if rows <= 4 else 8 if rows <= 8 else 16
    T = max(16 // RP, S)
    waves = -(-K // (32 if dtype == BF16 else 16) // (8 * T))                      # groups per wave
    return "float" if dtype == F32 else "unsigned short", S, RP, 2 if waves <= 2 or T // S == 4 else 4 if waves <= 4 else 8, 1


def test_every_residual_kernel_is_reached(lib):  # noqa: F811
    adds = lib["_ZN8sprinter14gemm_adds_rowsEiiii"]
    reached = set()
    for dtype in (F32, BF16):
        for d in WIDTHS:
            for rows in range(1, 41):
                for K in {d, 8, 264, 520, 1032, 2048, 4096, 4 * d, 32768}:
                    if _takes_norm(lib, dtype, d, rows) or adds(dtype, d, K, rows) & 0xFF:
                        reached.add(_resid_kernel(dtype, d, K, rows))
    compiled = _compiled(lib, "k_gemm_resid")
    # its accumulators hold every tile of a column only so
    assert all(16 // int(rp) >= int(s) or rp == "16" for _, _, s, rp, _, _ in compiled)
    assert compiled == {(t, arch, str(S), str(RP), str(UG), str(MT)) for t, S, RP, UG, MT in reached for arch in ("0", "1")}


@pytest.mark.parametrize("dtype, N, rows", [(BF16, 1600, 33), (BF16, 4096, 40), (F32, 512, 17), (F32, 2112, 1), (F32, 4096, 4)])
def test_products_without_a_kernel_are_refused(lib, dtype, N, rows):  # noqa: F811
    null = C.c_void_p(None)
    for arch in (0, 1):
        assert not lib[RESID](dtype, arch, null, null, N, 64, null, null, null, rows, null) & 0xFF


def test_every_kernel_with_the_norm_inside_is_reached(lib):  # noqa: F811
    reached = set()
    for dtype in (F32, BF16):
        for d in WIDTHS:
            for rows in range(1, 41):
                if not _takes_norm(lib, dtype, d, rows):
                    continue
                RG = 8 if d <= 512 else 4 if d <= 1024 else 2 if d <= 2048 else 1    # groups of 512 / RG threads of 8 columns
                RT = 1 if rows <= RG else 2 if rows <= 2 * RG else 4
                assert RT * RG >= rows and 4096 // RG >= d
                for tiles in (1, 2) if dtype == BF16 and 1024 < d <= 2048 else (1,):   # column tiles per wave
                    for arch in (0, 1):
                        for epi, emb in ((2 + arch, "false"), (0, "false"), (0, "true")):
                            reached.add(("float" if dtype == F32 else "unsigned short", str(arch), str(RT), str(RG), str(tiles), str(epi), emb))
    assert _compiled(lib, "k_norm_gemm") == reached


@pytest.mark.parametrize("dtype, d, rows", [(F32, 512, 17), (F32, 1024, 9), (F32, 2048, 5), (F32, 2112, 1), (BF16, 1024, 17), (BF16, 2048, 9), (BF16, 4096, 5), (BF16, 4160, 1)])
def test_norms_without_a_kernel_are_refused(lib, dtype, d, rows):  # noqa: F811
    """One row beyond each limit, and one column: nothing is launched, neither on fewer rows nor not at all without a word."""
    assert not _takes_norm(lib, dtype, d, rows)
    null = C.c_void_p(None)
    for arch in (0, 1):
        for epi in (0, 2 + arch):
            for N in (192, 8192):
                assert not lib[NORM_GEMM](dtype, arch, epi, null, null, null, null, C.c_float(1e-5), null, null, null, null, N, d, null, null, rows, null) & 0xFF


@pytest.mark.parametrize("dtype, d", [(F32, 64), (BF16, 64), (BF16, 4096)])
def test_longer_k_than_the_offsets_hold_stays_in_shares(lib, dtype, d):  # noqa: F811
    """d_ff has no limit of its own, and the buffers' sizes and offsets are 32 bits (16 float32 rows of 2^25 are 2^31 bytes)."""
    adds, null = lib["_ZN8sprinter14gemm_adds_rowsEiiii"], C.c_void_p(None)
    for K in ((1 << 20) + 8, 1 << 25, 1 << 28):
        assert not adds(dtype, d, K, 5) & 0xFF
        assert not lib[RESID](dtype, 0, null, null, d, K, null, null, null, 5, null) & 0xFF
