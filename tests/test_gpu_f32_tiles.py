"""The fp32 expert kernel against the oracle at the edges of its tiles: one
row, a full 16-row group, one over it, a full 64-row tile, one over it, over
reductions of one, odd and several 64-wide steps, with an always-on expert."""
import pytest

from tests import test_gpu_parity as P
from workload import make_accounts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,F,Fs", [(64, 64, 64), (192, 320, 0), (128, 256, 448)])
@pytest.mark.parametrize("T,mode", [(1, "eat"), (16, "topk"), (17, "topk"), (64, "eat"), (65, "eat"), (129, "topp")])
def test_f32_tiles(d, F, Fs, T, mode):
    c = dict(shape="tiny", d=d, F=F, E=8, Fs=Fs)
    shape, w, lay, prm = P._layer(c, mode, max_tokens=T)
    acc = make_accounts(8, seed=T, c_scale=0.05)
    P._forward_check(f"f32 d={d} F={F} {mode} T={T}", lay, shape, P._x_host(shape, T, d, seed=T + d), w, prm, acc=acc)
