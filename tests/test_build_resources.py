"""What the compiler says about the kernels (device code only, no GPU)."""
import os
import re
from concurrent.futures import ThreadPoolExecutor

from paper_2509_18085_amd import build


def test_no_matrix_core_kernel_uses_scratch_memory():
    """Every tile shape of every epilogue keeps its accumulators, fragments and epilogue values in registers: with scratch memory a
    kernel starts later and its epilogue waits for it."""
    sources = [s for s in build.SOURCES if s.startswith("mfma_")]
    assert len(sources) >= 7
    with ThreadPoolExecutor(max_workers=min(4, os.cpu_count() or 1)) as ex:
        for source, kernels in zip(sources, ex.map(build.scratch_bytes, sources)):
            assert not {k: n for k, n in kernels.items() if n}, source


def _sgprs(token):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", token)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    return {int(token[1:])} if re.fullmatch(r"s\d+", token) else set()


def _early_reads(text):
    """Vector memory instructions that read a scalar register less than five wait states after a vector instruction wrote it."""
    age, found = {}, []
    for line in text.splitlines():
        words = line.split(";")[0].replace(",", " ").split()
        if not words or words[0].endswith(":") or words[0].startswith("."):
            continue
        op, args = words[0], words[1:]
        if op.startswith(("global_", "buffer_", "flat_", "scratch_")) and any(age.get(r, 9) < 5 for a in args for r in _sgprs(a)):
            found.append(line.strip())
        step = int(args[0], 0) + 1 if op == "s_nop" else 1
        age = {r: n + step for r, n in age.items() if n + step < 5}
        if args and op.startswith(("v_readlane", "v_readfirstlane", "v_cmp")):
            age.update({r: 0 for r in _sgprs(args[0])})
        elif args and op.startswith("s_") and not op.startswith(("s_nop", "s_waitcnt", "s_cmp")):
            for r in _sgprs(args[0]):
                age.pop(r, None)
    return found


def test_no_transfer_reads_its_base_too_early():
    """The transfers into LDS are assembly with a scalar base, so the compiler does not keep them five wait states away from a
    vector instruction that writes the base (a scalar register that was parked in a vector register comes back that way)."""
    transfer = "s_mov_b32 m0, s9\ns_nop 0\nglobal_load_lds_dwordx4 v1, s[4:5]\n"
    assert _early_reads("v_readlane_b32 s5, v7, 3\n" + transfer)
    assert not _early_reads("v_readlane_b32 s5, v7, 3\ns_nop 2\n" + transfer)
    assert not _early_reads("v_readlane_b32 s5, v7, 3\ns_add_u32 s5, s5, s6\n" + transfer)
    sources = [s for s in build.SOURCES if s.startswith("mfma_") or s == "tile_gemm.hip"]
    with ThreadPoolExecutor(max_workers=min(4, os.cpu_count() or 1)) as ex:
        for source, text in zip(sources, ex.map(build.assembly, sources)):
            assert "global_load_lds_dwordx4" in text or source in ("mfma_gemm.hip",), source
            assert not _early_reads(text), (source, _early_reads(text)[:3])
