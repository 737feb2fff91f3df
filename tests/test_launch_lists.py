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


def _up(g):
    return next(n for n, _ in g["kernels"] if "stream_kernel<true" in n or "wide_kernel<true" in n)


def _tile(name):
    for tile, text in (("wide", "Tile<256, 256"), ("tall", "Tile<256, 128"), ("mid", "Tile<128, 128")):
        if text in name:
            return tile
    assert "stream_kernel" in name
    return "stream"


# (E, top_k, d_model, d_ffn), mode (0 EAT, 1 Top-K, 2 Top-P), tokens -> the kernel
# that measured faster there
MIXTRAL, FINE, QWEN = (8, 2, 4096, 14336), (64, 8, 2048, 1024), (128, 8, 2048, 768)
ROUTES = [(MIXTRAL, 0, 64, "stream"), (MIXTRAL, 0, 96, "mid"), (MIXTRAL, 0, 128, "mid"), (MIXTRAL, 0, 160, "tall"),
          (MIXTRAL, 0, 320, "mid"), (MIXTRAL, 0, 384, "mid"), (MIXTRAL, 0, 512, "tall"), (MIXTRAL, 0, 768, "tall"),
          (MIXTRAL, 2, 384, "mid"), (MIXTRAL, 2, 800, "tall"), (MIXTRAL, 1, 500, "tall"), (MIXTRAL, 1, 1024, "wide"),
          (FINE, 0, 65, "mid"), (FINE, 0, 256, "mid"), (FINE, 0, 320, "mid"), (FINE, 0, 384, "mid"),
          (FINE, 0, 1024, "tall"), (FINE, 2, 512, "mid"), (FINE, 2, 1024, "tall"), (FINE, 1, 768, "tall"),
          (QWEN, 0, 65, "stream"), (QWEN, 0, 96, "stream"), (QWEN, 0, 97, "mid"), (QWEN, 0, 384, "tall"),
          (QWEN, 0, 512, "tall"), (QWEN, 0, 640, "mid"), (QWEN, 1, 65, "mid"), (QWEN, 2, 1500, "tall")]


def test_medium_calls_take_the_faster_tile(tmp_path):
    """The up/gate kernel of calls of more than 64 tokens, the same for both
    weight layouts (which give the same bits)."""
    calls = [dict(kind="forward", T=T, mode=mode, E=s[0], top_k=s[1], d_model=s[2], d_ffn=s[3], top_p=0.6,
                  weight_layout=lay) for s, mode, T, _ in ROUTES for lay in (L.EAT_LAYOUT_ROWS, L.EAT_LAYOUT_PACKED)]
    got = list_launches(tmp_path, calls)
    for i, (s, mode, T, want) in enumerate(ROUTES):
        assert [_tile(_up(g)) for g in got[2 * i:2 * i + 2]] == [want] * 2, (s, mode, T)


def test_streaming_route_needs_no_more_workspace(tmp_path):
    """Calls of 65 to 96 tokens that go to the streaming kernel hold its gate/up
    partials where the down projection's slices go later: no call of that size
    that fits a given scratch on the tiles (one token more) stops fitting."""
    shapes = [(16, 4, 1024, 1024), (128, 8, 2048, 768), (64, 1, 512, 4096), (8, 1, 256, 7936), (32, 8, 192, 256),
              (128, 2, 4096, 256)]
    calls = [dict(kind="forward", T=T, mode=0, E=E, top_k=K, d_model=d, d_ffn=F) for E, K, d, F in shapes
             for T in (65, 80, 96, 97)]
    got = list_launches(tmp_path, calls)
    streams = 0
    for i in range(0, len(calls), 4):
        per = [g["bytes"] / c["T"] for g, c in zip(got[i:i + 4], calls[i:i + 4])]
        streams += _tile(_up(got[i])) == "stream"
        for g, c, b in zip(got[i:i + 4], calls[i:i + 4], per):
            # h and the slices of the down projection, the tiles' two large regions, and the rest
            assert b <= 1.03 * per[3], (c, per)
    assert streams >= 2


def test_head_just_over_a_round_of_tiles_streams(tmp_path):
    """The LM head of few sequences a little over 256 weight tiles of 128 rows
    (32768) would pay a second, nearly empty round on the tiles."""
    routes = [(1, 4096, 32768, "mid"), (1, 4096, 32832, "stream"), (64, 4096, 32000, "mid"), (32, 4096, 32832, "stream"),
              (1, 2048, 40000, "stream"), (64, 4096, 40000, "mid"), (1, 4096, 50304, "mid"), (96, 4096, 32832, "mid"),
              (1, 4096, 128256, "mid"), (129, 4096, 32832, "tall"), (384, 4096, 32832, "tall"), (384, 4096, 32768, "wide"),
              (3, 128, 64, "stream")]
    got = list_launches(tmp_path, [dict(kind="ppl", T=S, d=d, V=V) for S, d, V, _ in routes])
    for (S, d, V, want), g in zip(routes, got):
        name, (_, _, _, threads) = g["kernels"][0]
        assert _tile(name) == want, (S, d, V, name)
        # logits of two reduction slices at most
        assert 4 * S * V <= g["bytes"] <= 8 * S * V + 256
