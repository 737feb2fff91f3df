"""Calls of at most 256 tokens work out the token -> expert permutation inside
the up/gate launch: around every boundary of its 64-token groups and of the
64-expert mask words, in each of the three kernels that do it (fp32, streaming,
medium tiles), and one token above it, where the permutation is a launch."""
import pytest

from tests import test_gpu_parity as P
from workload import make_accounts

pytestmark = pytest.mark.gpu

CASES = {
    "f32_e64": dict(shape="tiny", d=64, F=64, E=64, Fs=0),
    "f32_e130": dict(shape="tiny", d=64, F=64, E=130, Fs=0),
    "e3": dict(shape="mixtral", d=192, F=192, E=3, Fs=0),
    "e64": dict(shape="finegrained", d=192, F=192, E=64, Fs=0),
    "e65": dict(shape="qwen3", d=192, F=192, E=65, Fs=0),
    "e256": dict(shape="qwen3", d=192, F=192, E=256, Fs=0),
    "short_e200": dict(shape="qwen3", d=128, F=128, E=200, Fs=0),     # streaming kernel at every size
}


@pytest.mark.parametrize("case", sorted(CASES))
@pytest.mark.parametrize("T,mode", [(1, "topp"), (63, "topk"), (64, "eat"), (65, "topk"), (128, "eat"), (129, "topk"),
                                    (193, "eat"), (255, "topk"), (256, "topp"), (257, "topk")])
def test_fused_permutation(case, T, mode):
    c = CASES[case]
    shape, w, lay, prm = P._layer(c, mode, K=min(P.SHAPES[c["shape"]].K, c["E"]), max_tokens=T)
    acc = make_accounts(c["E"], seed=T, c_scale=0.05)
    P._forward_check(f"permute {case} {mode} T={T}", lay, shape, P._x_host(shape, T, c["d"], seed=T), w, prm, acc=acc)


@pytest.mark.parametrize("E", [1, 8])
@pytest.mark.parametrize("T", [255, 256, 257])
@pytest.mark.parametrize("mode", ["eat", "topk", "topp"])
def test_top_k_of_every_expert(E, T, mode):
    """K = E: at 256 tokens the experts' average of 256 rows makes it a
    prefill-sized call, which takes the permutation launch."""
    c = dict(shape="mixtral", d=512, F=768, E=E, Fs=0)
    shape, w, lay, prm = P._layer(c, mode, K=E, max_tokens=T)
    acc = make_accounts(E, seed=T, c_scale=0.05)
    P._forward_check(f"permute K=E={E} {mode} T={T}", lay, shape, P._x_host(shape, T, c["d"], seed=T), w, prm, acc=acc)
