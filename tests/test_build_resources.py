"""What the compiler says about the kernels (device code only, no GPU)."""
import os
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
