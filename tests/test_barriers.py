"""The buffer-to-LDS loads written as inline assembly (dma16, dma4) are LDS writes
that the compiler does not see, and its barrier builtin does not order memory
accesses by itself: a kernel that uses them takes its barriers from dma_barrier,
across which no access may move. (The packed GEMMs choose per mode: the modes
with the builtin loads keep the builtin barrier.)"""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_23996_amd", "csrc")


def test_kernels_with_assembly_loads_use_the_ordering_barrier():
    seen = 0
    for name in sorted(os.listdir(CSRC)):
        if not name.endswith(".hip"):
            continue
        src = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, name)).read())
        for kernel in src.split("__global__")[1:]:
            if not re.search(r"\bdma(16|4)\(", kernel):
                continue
            seen += 1
            assert "dma_barrier();" in kernel, (name, kernel[:120])
            raw = len(re.findall(r"__builtin_amdgcn_s_barrier\(\)", kernel))
            chosen = len(re.findall(r"dma_barrier\(\);\s*else __builtin_amdgcn_s_barrier\(\)", kernel))
            assert raw == chosen, (name, kernel[:120])
    assert seen == 5  # attention, dW_gate, packed GEMMs, router logits, weight gradients
