"""Register budget of the latency-bound kernels (CPU; compiles for gfx950).

The one-launch block kernel, the fused MRConv and the in-register kNN run at
three waves per SIMD, the lean MRConv, the resident-key kNN and the direct-load
GEMM at four or more, the wide kNN and a small grid's MRConv at two; if the register allocator has to spill to scratch memory to
meet that, or gives a wave up, they slow down without failing any parity test.
This test compiles their sources with the resource-usage remarks and requires no
scratch, and the waves where they hang on registers alone, for every
instantiation of them."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_21290_amd", "csrc")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
KERNELS = {"block.hip": "block_kernel",
           "mrconv.hip": r"13mrconv_kernel|mrconv_lean_kernel|mrconv_cols_kernel|mr_gather_kernel",
           "knn.hip": "knn_kernel", "knn_wide.hip": "knn_wide_kernel",
           "knn_resident.hip": "knn_resident_kernel", "knn_stream.hip": "knn_stream_kernel",
           "gemm_dma.hip": "gemm_dma_kernel", "mlp.hip": "mlp_kernel"}
# where LDS holds more workgroups than registers do
WAVES = {"knn.hip": 3, "gemm_dma.hip": 4}


def _usage(src: str, tmp) -> list:
    out = os.path.join(str(tmp), src + ".o")
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-c",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-Rpass-analysis=kernel-resource-usage", os.path.join(CSRC, src), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    rows, name, scratch = [], None, 0
    for line in r.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
        m = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line)
        if m:
            scratch = int(m.group(1))
        m = re.search(r"Occupancy \[waves/SIMD\]: (\d+)", line)
        if m and name:
            rows.append((name, scratch, int(m.group(1))))
    return rows


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_latency_bound_kernels_do_not_spill(tmp_path):
    with ThreadPoolExecutor(len(KERNELS)) as ex:
        res = dict(zip(KERNELS, ex.map(lambda s: _usage(s, tmp_path), KERNELS)))
    for src, pat in KERNELS.items():
        ks = [r for r in res[src] if re.search(pat, r[0])]
        assert ks, f"no {pat} instantiation found in {src}"
        bad = [(n, sc) for n, sc, _ in ks if sc]
        assert not bad, f"{src}: kernels using scratch: {bad[:4]}"
        bad = [(n, occ) for n, _, occ in ks if occ < WAVES.get(src, 1)]
        assert not bad, f"{src}: kernels short of waves: {bad[:4]}"


def test_asm_names_the_m0_it_writes():
    """An asm statement that writes M0 lists it as clobbered: the compiler may hold
    a value of its own there (indexed moves, messages, LDS loads it makes itself)."""
    found = 0
    for name in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, name)) as f:
            text = f.read()
        for m in re.finditer(r"asm\s+volatile\s*\((.*?)\);", text, re.S):
            if re.search(r"\bs_mov_b32 m0\b|\bm0, ", m.group(1)):
                found += 1
                assert '"m0"' in m.group(1).rsplit(":", 1)[-1], (name, m.group(0))
    assert found
