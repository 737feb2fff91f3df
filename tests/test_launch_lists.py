"""What the host code launches, listed on the CPU (tests/launch_list.py)."""
import os
import shutil

import pytest

from paper_2609_33614_amd import _lib as L
from tests.launch_list import list_launches

pytestmark = pytest.mark.skipif(not os.path.exists(L.LIB_PATH) or shutil.which("g++") is None,
                                reason="needs libeat.so and g++")

# kernels that work the permutation out themselves: fp32, streaming, and the
# medium tiles of wide_kernel (128 weight rows; the prefill tile has 256)
FUSES = ("ffn_f32_kernel<true>", "stream_kernel<true", "Tile<256, 128", "Tile<128, 128")


def test_every_call_builds_its_permutation(tmp_path):
    """Each forward either launches the permutation or starts its experts with a
    kernel that works it out, never neither: over token counts around 256 (the
    most a fused call has) and every K up to E, whose largest values send
    calls of 256 tokens to the prefill tile."""
    calls = []
    for kind in ("forward", "noalloc", "stack"):
        for bf16 in ((1, 0) if kind != "stack" else (1,)):
            for d, F in ((512, 768), (256, 128), (192, 192), (128, 128)):
                for E, K in ((1, 1), (3, 3), (8, 8), (8, 7), (8, 2), (64, 64), (64, 1)):
                    for mode in ((0, 1, 2) if kind == "forward" else (0,)):
                        for T in (1, 64, 65, 128, 255, 256, 257, 512):
                            if kind == "noalloc" and E == 64 and T > 64:
                                continue          # more than its fixed scratch
                            calls.append(dict(kind=kind, T=T, mode=mode, E=E, top_k=K, d_model=d, d_ffn=F,
                                              act_dtype=bf16, expert_dtype=bf16))
    got = list_launches(tmp_path, [dict(c) for c in calls])
    assert len(got) == len(calls)
    wide = 0
    for c, g in zip(calls, got):
        names = [k for k, _ in g["kernels"]]
        layers = 2 if c["kind"] == "stack" else 1
        ups = [n for n in names if "ffn_f32_kernel<true>" in n or "stream_kernel<true" in n or "wide_kernel<true" in n]
        assert len(ups) == layers, (c, names)
        permutes = sum("permute_kernel" in n for n in names)
        fused = sum(any(f in n for f in FUSES) for n in ups) if c["T"] <= 256 else 0
        assert permutes + fused == layers, (c, names)
        wide += c["T"] == 256 and "Tile<256, 256" in ups[0]
    assert wide > 0                               # the calls where the two sizes meet are among them
